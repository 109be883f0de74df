// Small batches (internal): the search's stages before its scan in one launch,
// the tiles of the scans in another, and a direct scan without tiles.
//
// A search of a few queries is bound by launches (about 5.5 us each on this
// path, however little they do) and by the latency of kernels that leave the
// chip nearly empty.  The batch-sized path takes 19 launches for the plain scan
// and 35 for the pruning scan; with up to kSmallQ queries
//   k_front         one workgroup per query: filter, finite check, rounded
//                   query, centroid scores, best m partitions, sub-partitions
//   k_small_tiles   one workgroup per 64 partitions: the tiles of both scan rounds
// replace all of them but the scans and the merge, and where the batch's rows
// are few (direct_fits)
//   k_direct        one workgroup per (query, probe): filter, exact distances
//   k_direct_merge  one workgroup per query
// replace the scans too.  Results do not depend on the path.
#include <algorithm>

#include "caps_device.h"
#include "caps_internal.h"
#include "caps_mfma.h"
#include "caps_query.h"
#include "caps_small.h"

namespace caps {

constexpr int kFrontNT = 1024;
constexpr int kFrontNW = kFrontNT / 64;
constexpr int kBins = 2048;
constexpr int kRouteD = 16;              // dimensions per staged step
constexpr int kRouteS = kRouteD + 4;     // row stride of the staged step, in floats

// Exclusive scan over the kFrontNT threads (two barriers; `wsum` of kFrontNW).
__device__ inline int front_scan(int v, int *wsum) {
    const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
    const int inc = wave_incl_scan(v);
    __syncthreads();   // wsum is no longer read
    if (lane == 63) wsum[w] = inc;
    __syncthreads();
    int base = 0;
#pragma unroll
    for (int i = 0; i < kFrontNW; i++) base += i < w ? wsum[i] : 0;
    return base + inc - v;
}

// The need-th smallest of keys[0..b) under the order (key, index): taken are the
// keys below T and, of those equal to T, the indexes up to idl.  Histogram
// passes over 2^11 bins of the keys' own range [lo, hi], narrowed to the bin
// that holds the need-th key until that bin is taken whole or holds one value.
__device__ inline void front_kth(const uint32_t *keys, int b, int need, uint32_t lo, uint32_t hi, int32_t *hist,
                                 int *wsum, int *found, uint32_t &T, int &idl) {
    const int t = threadIdx.x;
    for (int pass = 0; pass < 4; pass++) {   // 32 bits, 11 per pass
        const uint32_t range = hi - lo;
        const int sh = range < (uint32_t)kBins ? 0 : 21 - __builtin_clz(range);
        hist[2 * t] = 0;
        hist[2 * t + 1] = 0;
        __syncthreads();
        for (int i = t; i < b; i += kFrontNT) {
            const uint32_t k = keys[i];
            if (k >= lo && k <= hi) atomicAdd(&hist[(k - lo) >> sh], 1);
        }
        __syncthreads();
        const int c0 = hist[2 * t], c1 = hist[2 * t + 1];
        const int pre = front_scan(c0 + c1, wsum);
        if (pre < need && need <= pre + c0 + c1) {   // one thread
            const bool second = need > pre + c0;
            found[0] = 2 * t + (second ? 1 : 0);
            found[1] = pre + (second ? c0 : 0);
            found[2] = second ? c1 : c0;
        }
        __syncthreads();
        const int bin = found[0], cnt = found[2];
        need -= found[1];
        lo += (uint32_t)bin << sh;
        hi = (uint32_t)min((uint64_t)hi, (uint64_t)lo + ((1ull << sh) - 1ull));
        if (cnt == need) {
            T = hi;
            idl = INT32_MAX;
            return;
        }
        if (sh == 0) break;
    }
    // more keys equal to lo than needed: the smallest indexes
    int run = 0;
    for (int i0 = 0; i0 < b; i0 += kFrontNT) {
        const int i = i0 + t;
        const int f = i < b && keys[i] == lo ? 1 : 0;
        const int at = run + front_scan(f, wsum);
        if (f && at == need - 1) found[3] = i;
        if (t == kFrontNT - 1) found[4] = at + f;
        __syncthreads();
        run = found[4];
    }
    T = lo;
    idl = found[3];
}

// One workgroup per query.  Routing: wave w scores centroids 64 w.. (then 1024
// on), one per lane; their rows come 16 dimensions at a time, coalesced, four
// steps ahead in registers, through a wave-private transposing tile in LDS (no
// workgroup barrier), and each lane sums its centroid's products in ascending
// order as k_scores_mfma does.  The best partitions are found by front_kth
// instead of a sort.  Latency bound: one query against 1024 x 128 centroids
// 14 us, against 22 us for scores, 20 us for the selection and six more
// launches on the batch-sized path.
template <bool VEC>
__global__ __launch_bounds__(kFrontNT) void k_front(FrontArgs A) {
    extern __shared__ __align__(16) unsigned char fsm[];
    uint32_t *keys = reinterpret_cast<uint32_t *>(fsm);                    // b
    float *qrow = reinterpret_cast<float *>(keys + ((A.b + 3) & ~3));      // d, zero padded to kRouteD
    const int dp = (A.d + kRouteD - 1) / kRouteD * kRouteD;
    float *tile = qrow + dp;                                               // kFrontNW x 64 x kRouteS
    int32_t *hist = reinterpret_cast<int32_t *>(tile);                     // kBins (after the routing)
    __shared__ int wsum[kFrontNW], found[5];
    __shared__ uint32_t wlo[kFrontNW], whi[kFrontNW];
    __shared__ QDesc qds, cur;
    __shared__ int nslot[2], ncand_s, bad_s;
    const int t = threadIdx.x, w = t >> 6, lane = t & 63;
    const int64_t q = blockIdx.x;
    const int b = A.b, d = A.d, m = A.m;
    const float *qg = A.q + q * d;
    for (int j = t; j < dp; j += kFrontNT) qrow[j] = j < d ? qg[j] : 0.0f;
    if (t == 0) {
        nslot[0] = nslot[1] = 0;
        ncand_s = 0;
        bad_s = 0;
        A.tau[q] = ~0ull;
        if (A.dcnt) A.dcnt[q] = 0;
        if (A.oflow) A.oflow[q] = 0;
        if (A.nsurv) A.nsurv[q] = 0;
        if (q == 0) A.cursor[0] = A.cursor[1] = 0;
    }
    __syncthreads();

    // ---- filter (wave 0) and query copy (wave 1), while the others score
    if (w == 0) {
        // (k_qprep's rules; one lane adds the pairs the wave has loaded)
        const int32_t lo = A.con_off[q], hi = A.con_off[q + 1];
        if (lane == 0) qd_clear(qds);
        if (lo < 0 || hi < lo || hi > A.n_con) {
            if (lane == 0) qds.flags |= kQUnsat;
        } else if (!A.disj) {
            for (int32_t e0 = lo; e0 < hi; e0 += 64) {
                const int32_t a = e0 + lane < hi ? A.con_attr[e0 + lane] : 0;
                const int32_t v = e0 + lane < hi ? A.con_val[e0 + lane] : 0;
                for (int i = 0; i < min(64, hi - e0); i++) {
                    const int32_t ai = __builtin_amdgcn_readlane(a, i), vi = __builtin_amdgcn_readlane(v, i);
                    if (lane == 0) qd_add(qds, A.sch, ai, vi);
                }
            }
        } else if (lane == 0) {
            qd_disjunction(qds, cur, A.qterms + q * kMaxTerms, A.sch, A.con_attr, A.con_val, lo, hi);
        }
    }
    if (w == 1) {
        bool ok = true;
        for (int j = lane; j < d; j += 64) ok &= __builtin_isfinite(qrow[j]);
        if (__ballot(!ok) != 0 && lane == 0) {
            bad_s = 1;
            atomicAdd(A.bad, 1);
        }
        if (A.qlow) qquant_row(qg, q, d, A.dpad, A.prec, true, A.qlow, A.qscale, A.qaux);
    }

    // ---- centroid scores
    {
        float *tl = tile + w * 64 * kRouteS;
        const int nst = dp / kRouteD;
        uint32_t klo = ~0u, khi = 0u;
        if (A.scores) {   // (pmask may share their memory: this row is read before it is written)
            for (int c = t; c < b; c += kFrontNT) {
                const uint32_t k = f2ord(A.scores[q * b + c]);
                keys[c] = k;
                klo = min(klo, k);
                khi = max(khi, k);
            }
        }
        for (int c0 = w * 64; c0 < b && !A.scores; c0 += kFrontNT) {
            const int lr = lane >> 2, lc = 4 * (lane & 3);
            float4 pf[4][4];
            auto load = [&](float4 (&v)[4], int s) {
#pragma unroll
                for (int i = 0; i < 4; i++) {
                    const int row = min(c0 + 16 * i + lr, b - 1), j = s * kRouteD + lc;
                    const float *src = A.cent + (int64_t)row * d + j;
                    if (VEC) {
                        v[i] = j < d ? *reinterpret_cast<const float4 *>(src) : make_float4(0.0f, 0.0f, 0.0f, 0.0f);
                    } else {
                        v[i] = make_float4(j < d ? src[0] : 0.0f, j + 1 < d ? src[1] : 0.0f, j + 2 < d ? src[2] : 0.0f,
                                           j + 3 < d ? src[3] : 0.0f);
                    }
                }
            };
#pragma unroll
            for (int u = 0; u < 4; u++)
                if (u < nst) load(pf[u], u);
            float acc = 0.0f;
            for (int s0 = 0; s0 < nst; s0 += 4) {
#pragma unroll
                for (int u = 0; u < 4; u++) {
                    const int s = s0 + u;
                    if (s >= nst) break;
                    wave_sync();   // the previous step is read
#pragma unroll
                    for (int i = 0; i < 4; i++)
                        *reinterpret_cast<float4 *>(tl + (16 * i + lr) * kRouteS + lc) = pf[u][i];
                    if (s + 4 < nst) load(pf[u], s + 4);
                    wave_sync();
#pragma unroll
                    for (int jj = 0; jj < kRouteD; jj += 4) {
                        const float4 cv = *reinterpret_cast<const float4 *>(tl + lane * kRouteS + jj);
                        const float4 qv = *reinterpret_cast<const float4 *>(qrow + s * kRouteD + jj);
                        acc = fmaf(qv.x, cv.x, acc);
                        acc = fmaf(qv.y, cv.y, acc);
                        acc = fmaf(qv.z, cv.z, acc);
                        acc = fmaf(qv.w, cv.w, acc);
                    }
                }
            }
            const int c = c0 + lane;
            if (c < b) {
                const uint32_t k = f2ord(canon0(A.metric == 0 ? A.cnorm[c] - 2.0f * acc : -acc));
                keys[c] = k;
                klo = min(klo, k);
                khi = max(khi, k);
            }
        }
#pragma unroll
        for (int o = 32; o >= 1; o >>= 1) {
            klo = min(klo, (uint32_t)__shfl_xor((int)klo, o, 64));
            khi = max(khi, (uint32_t)__shfl_xor((int)khi, o, 64));
        }
        if (lane == 0) {
            wlo[w] = klo;
            whi[w] = khi;
        }
    }
    __syncthreads();
    if (t == 0 && bad_s) qds.flags |= kQNonFinite;
    uint32_t lo = ~0u, hi = 0u;
#pragma unroll
    for (int i = 0; i < kFrontNW; i++) {
        lo = min(lo, wlo[i]);
        hi = max(hi, whi[i]);
    }
    // ---- the best m (and of them the best s, in the first slots); a NaN query
    // row makes NaN keys, in some order: its probes are never scanned
    uint32_t Tm, Ts = 0;
    int im, is = -1;
    const int s = A.s;
    front_kth(keys, b, m, lo, hi, hist, wsum, found, Tm, im);
    __syncthreads();
    if (s < m) {
        front_kth(keys, b, s, lo, hi, hist, wsum, found, Ts, is);
        __syncthreads();
    }
    if (t == 0) A.qd[q] = qds;
    int nc = 0;
    for (int i0 = 0; i0 < b; i0 += kFrontNT) {
        const int i = i0 + t;
        const uint32_t k = i < b ? keys[i] : ~0u;
        const bool in_m = i < b && (k < Tm || (k == Tm && i <= im));
        const bool in_s = in_m && s < m && (k < Ts || (k == Ts && i <= is));
        int r = 0;
        const uint64_t bs = __ballot(in_s), bm = __ballot(in_m && !in_s), lt = lanemask_lt();
        int base0 = 0, base1 = 0;
        if (lane == 0) {
            if (bs) base0 = atomicAdd(&nslot[0], __popcll(bs));
            if (bm) base1 = atomicAdd(&nslot[1], __popcll(bm));
        }
        base0 = __builtin_amdgcn_readfirstlane(base0);
        base1 = __builtin_amdgcn_readfirstlane(base1) + (s < m ? s : 0);
        r = in_s ? base0 + __popcll(bs & lt) : base1 + __popcll(bm & lt);
        uint32_t pm = 0;
        if (in_m && r < m) {
            const uint32_t mask = choose_query_levels(A.sch, qds, A.qterms + q * kMaxTerms, A.tags + (int64_t)i * A.h,
                                                      A.h, A.rule);
            int32_t cand = 0;
            for (int j = 0; j <= A.h; j++)
                if (mask & (1u << j)) cand += A.offs[(int64_t)i * (A.h + 1) + j + 1] - A.offs[(int64_t)i * (A.h + 1) + j];
            const int64_t e = q * m + r;
            A.probes[e] = i;
            A.sel[e] = mask;
            A.cand[e] = cand;
            nc += cand;
            if (mask) pm = mask | ((uint32_t)r << 16) | (in_s || s >= m ? kSmallSeed : 0u);
        }
        if (A.pmask && i < b) A.pmask[q * b + i] = pm;
    }
#pragma unroll
    for (int o = 32; o >= 1; o >>= 1) nc += __shfl_xor(nc, o, 64);
    if (lane == 0 && nc) atomicAdd(&ncand_s, nc);
    __syncthreads();
    if (t == 0) A.ncand[q] = ncand_s;
}

static size_t front_lds(const FrontArgs &A) {
    const size_t dp = (size_t)(A.d + kRouteD - 1) / kRouteD * kRouteD;
    return 4 * ((size_t)((A.b + 3) & ~3) + dp + (size_t)kFrontNW * 64 * kRouteS);
}

caps_status small_front(const FrontArgs &A, int32_t nq, int device, hipStream_t st) {
    const size_t lds = front_lds(A);
    const auto fn = A.d % 4 == 0 ? k_front<true> : k_front<false>;
    const caps_status ls = set_kernel_lds((const void *)fn, lds, device);
    if (ls != CAPS_OK) return ls;
    hipLaunchKernelGGL(fn, dim3((unsigned)nq), dim3(kFrontNT), lds, st, A);
    CAPS_HIP(hipGetLastError());
    return CAPS_OK;
}

bool small_fits(int32_t b, int32_t d, int32_t nq) { return nq <= kSmallQ && d <= 4096 && b <= kMaxPartitions; }

// ------------------------------------------------------------------ tiles
// Tiles of one or two scan rounds from the per-(query, partition) words.  Each
// partition takes its entries' place in a round's list from a cursor (cleared
// by k_front), in any order; a partition without entries has empty tiles.
// Each tile is written `split` times, for as many workgroups to share its rows.
// The tiles of an XCD's partitions follow each other first tiles first: most
// partitions fill one of their ceil(nq / qb), and with a partition's own next to
// each other the full ones of an XCD fell to every second or fourth compute unit
// only (226 queries, 83 partitions, seed pass 0.99 ms against 0.58).
// 64 partitions per workgroup of 16 waves, staged through LDS (the words are
// read by query, used by partition); one cursor access per workgroup and round
// (one per partition, each awaited, took 33 us for 24 queries).
constexpr int kTilesNT = 1024;
__global__ __launch_bounds__(kTilesNT) void k_small_tiles(const uint32_t *__restrict__ pmask, int32_t nq, int32_t b,
                                                          int32_t m, SmallRound R0, SmallRound R1,
                                                          int32_t *__restrict__ cursor) {
    extern __shared__ uint32_t pms[];   // nq x 65
    __shared__ int32_t cnt[2][64], at0[2][64];
    const int t = threadIdx.x, w = t >> 6, lane = t & 63, p0 = blockIdx.x * 64;
    for (int e = t; e < nq * 64; e += kTilesNT) {
        const int qi = e >> 6, pi = e & 63;
        pms[qi * 65 + pi] = p0 + pi < b ? pmask[(int64_t)qi * b + p0 + pi] : 0u;
    }
    __syncthreads();
    // which of the queries of 64-query group g have an entry of the round in
    // partition p0 + pi
    auto members = [&](int pi, int g, const SmallRound &R) {
        const int qi = g * 64 + lane;
        const uint32_t v = qi < nq ? pms[qi * 65 + pi] : 0u;
        return __ballot(v != 0 && (R.which == 0 || ((v & kSmallSeed) != 0) == (R.which == 1)));
    };
    const int ng = (nq + 63) / 64;
    for (int i = 0; i < 4; i++) {
        const int pi = w * 4 + i;
        for (int round = 0; round < 2; round++) {
            const SmallRound &R = round ? R1 : R0;
            int n = 0;
            for (int g = 0; g < ng; g++) n += __popcll(members(pi, g, R));
            if (lane == 0) cnt[round][pi] = R.entries ? n : 0;
        }
    }
    __syncthreads();
    if (w < 2) {
        const int n = cnt[w][lane];
        const int inc = wave_incl_scan(n);
        int base = 0;
        if (lane == 63 && inc) base = atomicAdd(cursor + w, inc);
        at0[w][lane] = __shfl(base, 63, 64) + inc - n;
    }
    __syncthreads();
    const uint64_t lt = lanemask_lt();
    for (int i = 0; i < 4; i++) {
        const int pi = w * 4 + i, p = p0 + pi;
        if (p >= small_padded(b)) break;
        for (int round = 0; round < 2; round++) {
            const SmallRound &R = round ? R1 : R0;
            if (!R.entries) continue;
            const int base = at0[round][pi], n = cnt[round][pi];
            int run = base;
            for (int g = 0; g < ng && n; g++) {
                const uint64_t bal = members(pi, g, R);
                if ((bal >> lane) & 1ull) {
                    const int qi = g * 64 + lane;
                    const uint32_t v = pms[qi * 65 + pi];
                    const int64_t at = run + __popcll(bal & lt);
                    R.entries[at] = qi * m + (int32_t)((v >> 16) & 0x1FFFu);
                    if (R.esel) R.esel[at] = v & 0xFFFFu;
                }
                run += __popcll(bal);
            }
            const int nt = (nq + R.qb - 1) / R.qb;   // tiles per partition
            const int px = small_padded(b) / kXcds, x = p / px;   // partitions of an XCD
            for (int i = lane; i < nt * R.split; i += 64) {
                const int ti = i / R.split, s = i - ti * R.split;
                R.tiles[((int64_t)(x * nt + ti) * px + (p - x * px)) * R.split + s] =
                    make_int4(p, base + ti * R.qb, max(0, min(R.qb, n - ti * R.qb)), s | (R.split << 8));
            }
        }
    }
}

caps_status small_tiles(const uint32_t *pmask, int32_t nq, int32_t b, int32_t m, const SmallRound &r0,
                        const SmallRound &r1, int32_t *cursor, int device, hipStream_t st) {
    const size_t lds = sizeof(uint32_t) * 65 * (size_t)nq;
    // (the largest batch's, once: a setting costs 0.2 ms, and batch sizes vary)
    const caps_status ls = set_kernel_lds((const void *)k_small_tiles, sizeof(uint32_t) * 65 * kSmallQ, device);
    if (ls != CAPS_OK) return ls;
    hipLaunchKernelGGL(k_small_tiles, dim3((unsigned)((b + 63) / 64)), dim3(kTilesNT), lds, st, pmask, nq, b, m, r0, r1,
                       cursor);
    CAPS_HIP(hipGetLastError());
    return CAPS_OK;
}

// ------------------------------------------------------------------ direct scan
// One workgroup per (query, probe): its threads filter the rows of the chosen
// sub-partitions (256 at a time, four loads each in flight), the rows that
// pass queue per wave and are scored exactly, one per lane (the plain scan's
// arithmetic); each wave keeps its best k, the workgroup writes the best k of
// them.  No reuse of rows between queries, so for few rows only: bytes of the
// rows that pass, 4 d each, and latency; one query over 64 probes of 976 rows
// in 9 us, against 16 + 7 + 18 us for the seed round and the pruning scan.
constexpr int kDirBuf = 128;

__global__ __launch_bounds__(256) void k_direct(DirectArgs A) {
    __shared__ uint64_t buf[4][kDirBuf], pool[4 * kMaxK];
    __shared__ uint32_t ring[4][128];
    __shared__ int32_t bcnt[4], pn;
    __shared__ uint64_t tau[4], ptau;
    __shared__ QDesc qds;
    __shared__ int32_t lst[kMaxHeight + 1], len[kMaxHeight + 2];   // chosen levels: first row, rows before
    const int64_t slot = blockIdx.x;
    const int t = threadIdx.x, w = t >> 6, lane = t & 63;
    const uint32_t sm = A.sel[slot];
    uint64_t *out = A.partials + slot * A.k;
    if (!sm) {   // (no barrier was passed)
        if (t < A.k) out[t] = ~0ull;
        return;
    }
    const int32_t qq = (int32_t)(slot / A.m);
    const int32_t p = A.probes[slot];
    if (t < 64) {
        bool on = t <= A.h && ((sm >> t) & 1u);
        const int32_t lo = on ? A.offs[(int64_t)p * (A.h + 1) + t] : 0;
        const int32_t n = on ? A.offs[(int64_t)p * (A.h + 1) + t + 1] - lo : 0;
        const int inc = wave_incl_scan(n);
        if (t <= A.h) {
            lst[t] = lo - (inc - n);   // CSR position of flat row f of level t: lst[t] + f
            len[t + 1] = inc;
        }
        if (t == 0) len[0] = 0;
    }
    if (t == 64) qds = A.qd[qq];
    if (t < 4) {
        bcnt[t] = 0;
        tau[t] = ~0ull;
    }
    if (t == 0) pn = 0;
    __syncthreads();
    const int total = len[A.h + 1];
    const bool has_dense = A.words != nullptr, has_lab = A.sigs != nullptr, is_or = (qds.flags & kQOr) != 0;
    const uint32_t dm = qds.dmask, dv = qds.dval;
    const uint64_t lsig = qds.lsig;
    const float *qr = A.q + (int64_t)__builtin_amdgcn_readfirstlane(qq) * A.d;
    const bool l2 = A.metric == 0;
    int head = 0, tail = 0, nsurv = 0;   // wave-uniform
    auto process = [&](int n) {
        wave_sync();
        bool v = lane < n;
        const uint32_t pos = v ? ring[w][(tail + lane) & 127] : 0u;
        tail += n;
        if (v && (is_or || (has_lab && qds.nlab > 0)))
            v = query_passes(qds, A.qterms + (int64_t)qq * kMaxTerms, has_dense, has_lab, has_dense ? A.words[pos] : 0u,
                             has_lab ? A.sigs[pos] : 0ull, has_lab ? A.slots + (int64_t)pos * A.lslots : nullptr,
                             A.lslots);
        nsurv += __popcll(__ballot(v));
        uint64_t key = ~0ull;
        if (v) {
            const float sc = exact_score<8>(A.vecs + (int64_t)pos * A.d, qr, A.d, l2);
            key = ((uint64_t)f2ord(sc) << 32) | (uint32_t)A.perm[pos];
        }
        const bool qual = v && key < tau[w];
        const uint64_t bal = __ballot(qual);
        if (!bal) return;
        if (bcnt[w] + __popcll(bal) > kDirBuf) buf_reduce<kDirBuf>(&buf[0][0], bcnt, tau, w, A.k);   // (k <= 64 remain)
        const int c = bcnt[w];
        if (qual) buf[w][c + __popcll(bal & lanemask_lt())] = key;
        wave_sync();
        if (lane == 0) bcnt[w] = c + __popcll(bal);
        wave_sync();
    };
    for (int f0 = 0; f0 < total; f0 += 1024) {
        int32_t pos[4];
        uint32_t wd[4];
        uint64_t sg[4];
        bool ok[4];
#pragma unroll
        for (int u = 0; u < 4; u++) {
            const int f = f0 + 256 * u + t;
            ok[u] = f < total;
            pos[u] = 0;
            for (int j = 0; j <= A.h; j++)
                if (f >= len[j] && f < len[j + 1]) pos[u] = lst[j] + f;
            wd[u] = has_dense && ok[u] ? A.words[pos[u]] : 0u;
            sg[u] = has_lab && ok[u] ? A.sigs[pos[u]] : 0ull;
        }
#pragma unroll
        for (int u = 0; u < 4; u++) {
            // (a disjunction's summary holds the dense fields its terms share and no labels)
            const bool pass = ok[u] && (wd[u] & dm) == dv && (lsig & ~sg[u]) == 0;
            const uint64_t bal = __ballot(pass);
            if (!bal) continue;
            if (pass) ring[w][(head + __popcll(bal & lanemask_lt())) & 127] = (uint32_t)pos[u];
            head += __popcll(bal);
            if (head - tail >= 64) process(64);
        }
    }
    if (head > tail) process(head - tail);
    buf_reduce<kDirBuf>(&buf[0][0], bcnt, tau, w, A.k);
    if (A.nsurv && lane == 0 && nsurv) atomicAdd(&A.nsurv[qq], nsurv);
    // the waves' lists, joined
    int base = 0;
    if (lane == 0) base = atomicAdd(&pn, bcnt[w]);
    base = __builtin_amdgcn_readfirstlane(base);
    if (lane < bcnt[w]) pool[base + lane] = buf[w][lane];
    __syncthreads();
    if (w == 0) {
        if (lane == 0) ptau = ~0ull;
        wave_sync();
        buf_reduce<4 * kMaxK>(pool, &pn, &ptau, 0, A.k);
        const int n = pn;
        if (lane < A.k) out[lane] = lane < n ? pool[lane] : ~0ull;
    }
}

// One workgroup per query: the best k of its m lists of k keys (padded with
// ~0), read as one run; each wave keeps its best k in an LDS pool.
__global__ __launch_bounds__(256) void k_direct_merge(const uint64_t *__restrict__ partials, int32_t m, int32_t k,
                                                      int32_t metric, int32_t *__restrict__ ids,
                                                      float *__restrict__ dist) {
    __shared__ uint64_t pool[4][256], fin[256];
    __shared__ int32_t np[4], fn;
    __shared__ uint64_t tau[4], ftau;
    const int64_t q = blockIdx.x;
    const int t = threadIdx.x, w = t >> 6, lane = t & 63;
    if (t < 4) {
        np[t] = 0;
        tau[t] = ~0ull;
    }
    if (t == 0) {
        fn = 0;
        ftau = ~0ull;
    }
    __syncthreads();
    const int64_t total = (int64_t)m * k;
    const uint64_t *src = partials + q * total;
    for (int64_t f0 = 0; f0 < total; f0 += 1024) {
        uint64_t key[4];
#pragma unroll
        for (int u = 0; u < 4; u++) {
            const int64_t f = f0 + 256 * u + t;
            key[u] = f < total ? src[f] : ~0ull;
        }
#pragma unroll
        for (int u = 0; u < 4; u++) {
            const bool has = key[u] < tau[w];   // (tau starts at ~0: padding never enters)
            const uint64_t bal = __ballot(has);
            if (!bal) continue;
            if (np[w] + 64 > 256) buf_reduce<256>(&pool[0][0], np, tau, w, k);
            const int c = np[w];
            if (has) pool[w][c + __popcll(bal & lanemask_lt())] = key[u];
            wave_sync();
            if (lane == 0) np[w] = c + __popcll(bal);
            wave_sync();
        }
    }
    buf_reduce<256>(&pool[0][0], np, tau, w, k);
    int base = 0;
    if (lane == 0) base = atomicAdd(&fn, np[w]);
    base = __builtin_amdgcn_readfirstlane(base);
    if (lane < np[w]) fin[base + lane] = pool[w][lane];
    __syncthreads();
    if (w != 0) return;
    buf_reduce<256>(fin, &fn, &ftau, 0, k);
    const int n = fn;
    if (lane < k) {
        const int64_t o = q * k + lane;
        const uint64_t best = lane < n ? fin[lane] : ~0ull;
        if (best == ~0ull) {
            ids[o] = -1;
            dist[o] = metric == 0 ? __builtin_huge_valf() : -__builtin_huge_valf();
        } else {
            ids[o] = (int32_t)(uint32_t)(best & 0xFFFFFFFFu);
            const float key = ord2f((uint32_t)(best >> 32));
            dist[o] = metric == 0 ? key : canon0(-key);
        }
    }
}

caps_status small_direct(const DirectArgs &A, int32_t nq, int32_t *ids, float *dist, hipStream_t st) {
    prof_begin(CAPS_STAGE_SCAN, st);
    hipLaunchKernelGGL(k_direct, dim3((unsigned)((int64_t)nq * A.m)), dim3(256), 0, st, A);
    prof_end(CAPS_STAGE_SCAN, st);
    prof_begin(CAPS_STAGE_MERGE, st);
    hipLaunchKernelGGL(k_direct_merge, dim3((unsigned)nq), dim3(256), 0, st, (const uint64_t *)A.partials, A.m, A.k,
                       A.metric, ids, dist);
    prof_end(CAPS_STAGE_MERGE, st);
    CAPS_HIP(hipGetLastError());
    return CAPS_OK;
}

// Rows the direct scan may have to score: at most 64M elements (every row of
// the batch's probes passing, 256 MB, takes about as long as the launches
// saved; at the benchmark's selectivities 1 in 16 passes).
bool direct_fits(const IndexData *ix, int32_t nq, int32_t m) {
    const double rows = (double)nq * m * ((double)ix->n / ix->b);
    return rows * ix->d <= 64e6 && (int64_t)nq * m <= (1 << 20);
}

}  // namespace caps
