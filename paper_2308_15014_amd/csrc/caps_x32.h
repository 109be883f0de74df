// Matrix-core scan on 32 x 32 blocks (internal): the exact main pass and the
// seed pass of rows of at most four 32-element steps (128 elements), in every
// storage format, with and without label tests and disjunctions.
// Instantiated by caps_x32_inst.hip.
//
// Same bound, point term and element test as k_scan_mfma's exact main pass;
// what differs is the blocking:
//  * a tile holds up to 128 (query, probe) entries of one partition, wave w
//    the 32 queries 32w..32w+31, whose operands stay in registers;
//  * each product is a 32 x 32 block (points x queries, K = 16 per step), so
//    a staged row read from LDS serves 32 queries instead of 16;
//  * chunks are 32 rows, staged by direct loads three chunks ahead into four
//    buffers, with explicit per-wave wait counts and plain barriers;
//  * the packed dense test runs only for the products where a score passed,
//    the label signature test and a disjunction's terms' dense fields and
//    signatures (staged data and registers) only where that passed too.  The
//    main pass makes the rest of the filter test (label slots; global reads)
//    when it drains a wave's ring of pairs, one pair per lane, so that one round trip to memory
//    serves up to 64 pairs; a pair was tested as it was found before, one
//    round trip for each block of products with any passing score.
// Element r of lane l is point 8(r/4) + 4(l/32) + r%4 of the chunk and query
// l%32 of the wave.  MODE 0 is the exact main pass, MODE 1 the same counting
// the survivors of the filter, MODE 2 the seed pass of the exact search:
// approximate keys (plain point term) of the first probes, of which each
// lane keeps its MH best that pass the filter in registers, written as the
// (query, probe)'s partial list for the seed bound; MODE 3 is the main pass of
// the approximate search: the plain point term, pairs at or below the query's
// bound on its r-th approximate key deferred with their approximate scores.
//
// An FP8 row's 32-element block is read as one 16-byte operand per lane like
// a two-byte row's 16-element step and multiplied as two K = 16 products (low
// and high halves): queries and points use the same order of the elements,
// and a dot product does not depend on it beyond its rounding, which the
// bound's margin covers for any order.
#pragma once

#include "caps_mfma.h"

namespace caps {

constexpr int kXW = 4;                 // waves per tile
constexpr int kXQ = 32;                // queries per wave
constexpr int kXQB = kXW * kXQ;        // entries per tile
constexpr int kXCH = 32;               // rows per chunk
constexpr int kXRing = 64;             // per-wave ring of deferred pairs
typedef float f32x16 __attribute__((ext_vector_type(16)));

// The product of one 16-byte operand of each side (16 elements of a row per
// half wave in the two-byte formats, 32 in FP8).
template <int PREC>
__device__ inline f32x16 mma32(uint4 a, uint4 b, f32x16 c) {
    if constexpr (PREC == CAPS_PREC_BF16) {
        return __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, a), __builtin_bit_cast(bf16x8, b), c,
                                                       0, 0, 0);
    } else if constexpr (PREC == CAPS_PREC_FP16) {
        return __builtin_amdgcn_mfma_f32_32x32x16_f16(__builtin_bit_cast(f16x8, a), __builtin_bit_cast(f16x8, b), c, 0,
                                                      0, 0);
    } else {
        const long a0 = (long)(((uint64_t)a.y << 32) | a.x), a1 = (long)(((uint64_t)a.w << 32) | a.z);
        const long b0 = (long)(((uint64_t)b.y << 32) | b.x), b1 = (long)(((uint64_t)b.w << 32) | b.z);
        c = __builtin_amdgcn_mfma_f32_32x32x16_fp8_fp8(a0, b0, c, 0, 0, 0);
        return __builtin_amdgcn_mfma_f32_32x32x16_fp8_fp8(a1, b1, c, 0, 0, 0);
    }
}

// Register budget per SIMD: four waves; three with the label state.
template <int PREC, int NS, int MODE, int MH, int FILT>
__global__ __launch_bounds__(kXW * 64) __attribute__((amdgpu_waves_per_eu(FILT ? 3 : 4))) void k_scan_x32(LowpArgs A) {
    constexpr bool LAB = FILT != 0;     // label tests (an index with labels)
    constexpr bool DISJ = FILT == 2;    // and disjunctions, on any index
    static_assert(!(LAB && MODE == 1), "survivors of label tests are counted by k_scan_mfma");
    constexpr bool COUNT = MODE == 1;   // survivor counts of the exact filter
    constexpr bool SEED = MODE == 2;    // approximate keys: per query and probe the best 2 MH
    constexpr bool APPROX = MODE >= 2;  // approximate scores (no margin)
    constexpr bool F8 = PREC == CAPS_PREC_FP8;
    constexpr int ROWB = NS * (F8 ? 32 : 64);      // bytes per row of the copy
    constexpr int KS = ROWB / 32;                  // 16-byte operands per lane and row
    constexpr bool PTS2 = LAB || F8;               // a second per-point load: signatures, FP8 scales
    constexpr int V16 = ROWB / 16;                 // 16-byte pieces per row
    constexpr int NDMA = kXCH * ROWB / 1024;       // 1 KB direct loads per chunk
    constexpr int UPW = (NDMA + kXW - 1) / kXW;
    constexpr int RPL = ROWB >= 256 ? 1 : 256 / ROWB;
    constexpr int SWZ = ROWB >= 256 ? 15 : V16 - 1;
    constexpr int PRE = 4;                         // per-point inputs per chunk (one direct load per wave)
    static_assert(PRE == kXW, "each wave stages one per-point input");
    // the four chunk buffers: distinct arrays, so that the compiler can tell
    // the reads of one from the direct loads into the others
    __shared__ __align__(16) uint8_t xb0[kXCH * ROWB];
    __shared__ __align__(16) uint8_t xb1[kXCH * ROWB];
    __shared__ __align__(16) uint8_t xb2[kXCH * ROWB];
    __shared__ __align__(16) uint8_t xb3[kXCH * ROWB];
    __shared__ __align__(16) float rw0[PRE][kXCH];   // the per-point inputs of each buffer's chunk
    __shared__ __align__(16) float rw1[PRE][kXCH];
    __shared__ __align__(16) float rw2[PRE][kXCH];
    __shared__ __align__(16) float rw3[PRE][kXCH];
    // the second per-point load: label signatures (two words each), FP8 scales
    __shared__ __align__(16) uint32_t rg0[PTS2 ? 3 : 1][PTS2 ? kXCH : 1];
    __shared__ __align__(16) uint32_t rg1[PTS2 ? 3 : 1][PTS2 ? kXCH : 1];
    __shared__ __align__(16) uint32_t rg2[PTS2 ? 3 : 1][PTS2 ? kXCH : 1];
    __shared__ __align__(16) uint32_t rg3[PTS2 ? 3 : 1][PTS2 ? kXCH : 1];
    typedef uint32_t (*Raw2)[PTS2 ? kXCH : 1];
    __shared__ __align__(16) uint64_t xsig[LAB ? 2 : 1][LAB ? kXCH : 1];   // signatures of the scored chunk
    __shared__ __align__(16) float xsc[F8 ? 2 : 1][F8 ? kXCH : 1];         // FP8 scales of the scored chunk
    // seed pass: the label slots of narrow rows (8 of them), beside the rows of each buffer
    constexpr bool SLOTS = SEED && LAB;
    __shared__ __align__(16) uint16_t xl0[SLOTS ? kXCH * kMaxLabels : 1];
    __shared__ __align__(16) uint16_t xl1[SLOTS ? kXCH * kMaxLabels : 1];
    __shared__ __align__(16) uint16_t xl2[SLOTS ? kXCH * kMaxLabels : 1];
    __shared__ __align__(16) uint16_t xl3[SLOTS ? kXCH * kMaxLabels : 1];
    __shared__ __align__(16) QDesc qds[LAB ? kXQB : 1];                    // the tile's filter descriptors
    __shared__ __align__(16) uint32_t xw[2][kXCH];
    __shared__ __align__(16) float xn[2][kXCH];
    __shared__ uint32_t xsum[2][2];   // AND and OR of each point slot's packed words (the chunk's rows)
    __shared__ uint32_t ring[kXW][SEED ? 2 : 3][kXRing];
    __shared__ int32_t dhist[kXW][kXQ];   // (before the pipeline starts: also the tile's maxima, below)
    __shared__ int32_t scnt[COUNT ? kXQB : 1];   // (only the counting mode: the modes used per search keep 4 workgroups per CU)
    // the tile prologue's per-wave maxima share the drain histograms' storage:
    // every read of them completes before the pipeline's first barrier, and
    // no drain runs before it
    static_assert(3 * kXW <= kXQ, "the maxima fit in one wave's histogram");
    float(*qmx)[kXW] = reinterpret_cast<float(*)[kXW]>(&dhist[0][0]);
    uint32_t *lvw = reinterpret_cast<uint32_t *>(&dhist[0][2 * kXW]);

    const int tile = xcd_tile(blockIdx.x, A.ntiles);
    if (tile < 0) return;
    const int4 dsc = A.tiles[tile];
    if (dsc.z <= 0) return;
    const int p = dsc.x;
    const int nqt = dsc.z;
    const int32_t *ent = A.entries + dsc.y;
    const int h = A.h;
    // the tile's share of the rows: chunks share, share + nshare, ... (small
    // batches; a whole tile has w = 0)
    const int share = dsc.w & 255, nshare = max(1, dsc.w >> 8);
    const int t = threadIdx.x, lane = t & 63;
    const int w = __builtin_amdgcn_readfirstlane(t >> 6);   // (wave-uniform: kept in a scalar register)
    const int g = lane >> 5, c32 = lane & 31;
    const bool has_dense = A.words != nullptr;
    const bool has_lab = LAB && A.sigs != nullptr;
    const bool narrow = SLOTS && has_lab && A.lslots == kMaxLabels;
    const bool l2 = A.metric == 0;
    const float qnan = __builtin_nanf("");
    const float inf = __builtin_huge_valf();
    const float cm = l2 ? -2.0f : -1.0f;   // score = cm * dot + per-point term

    // ---- the lane's query: tile entry 32w + c32 (lanes l and l + 32 share it)
    const int qi = kXQ * w + c32;
    const bool own = qi < nqt;
    int32_t my_slot = 0, my_qq = 0;
    uint32_t my_sel = 0, my_mask = 0, my_val = 1;   // a lane without a query never matches
    float my_tf = qnan, qa = 0.0f, qb = 0.0f;
    uint64_t my_tk = ~0ull;   // seed: the shared bound key at the tile's start
    uint64_t my_lsig = 0;     // signature bits of the query's label constraints
    bool my_or = false;       // the query is a disjunction: its terms' dense fields and signatures
    uint32_t tm[DISJ ? kMaxTerms : 1], tv[DISJ ? kMaxTerms : 1];
    uint64_t tl[DISJ ? kMaxTerms : 1];
#pragma unroll
    for (int i = 0; i < (DISJ ? kMaxTerms : 1); i++) {   // (a term that is not there never matches)
        tm[i] = 0;
        tv[i] = 1;
        tl[i] = 0;
    }
    float my_qs = 1.0f;       // FP8 scale of the query
    if (own) {
        my_slot = ent[qi];
        my_qq = my_slot / A.m;
        my_sel = A.esel ? A.esel[dsc.y + qi] : A.sel[my_slot];   // (in entry order: one coalesced read)
        if constexpr (LAB) {
            const QDesc qd = A.qd[my_qq];
            my_mask = qd.dmask;
            my_val = qd.dval;
            my_lsig = qd.lsig;
            my_or = DISJ && (qd.flags & kQOr) != 0;
            if (g == 0) qds[qi] = qd;   // (read by this wave only)
            if (DISJ && my_or) {
#pragma unroll
                for (int i = 0; i < kMaxTerms; i++) {
                    if (i >= qd.nterm) break;
                    const QDesc &td = A.qterms[(int64_t)my_qq * kMaxTerms + i];
                    tm[i] = td.dmask;
                    tv[i] = td.dval;
                    tl[i] = td.lsig;
                }
            }
        } else {
            my_mask = A.qd[my_qq].dmask;
            my_val = A.qd[my_qq].dval;
        }
        if (F8) my_qs = A.qscale[my_qq];
        const float4 ax = *reinterpret_cast<const float4 *>(A.qaux + 4 * (int64_t)my_qq);
        qa = ax.x;
        qb = fmaf(A.gam, ax.w, ax.z);
        // the bound, read once per tile (the main pass keeps no keys; the
        // seed pass shares it between the tiles of a query by atomic min)
        const uint64_t tk = __hip_atomic_load(A.tau + my_qq, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        const float td = bound_score(tk);
        const float nq = ax.y;
        my_tf = APPROX        ? td
                : !(td < inf) ? inf
                : l2          ? fmaf(A.eta, nq + td, td - nq) + 1e-37f
                              : fmaf(A.eta, nq + fabsf(td), td) + 1e-37f;
        if (SEED) my_tk = tk;
    }
    // tile maxima of |q| and |q - q~| + gam |q~| (the point term's error
    // products) and the levels any query of the tile selects
    uint32_t lv = my_sel;
#pragma unroll
    for (int o = 32; o >= 1; o >>= 1) {
        qa = fmaxf(qa, __shfl_xor(qa, o, 64));
        qb = fmaxf(qb, __shfl_xor(qb, o, 64));
        lv |= __shfl_xor(lv, o, 64);
    }
    if (lane == 0) {
        qmx[0][w] = qa;
        qmx[1][w] = qb;
        lvw[w] = lv;
    }
    if constexpr (COUNT) {
        if (w == 0) {
            scnt[lane] = 0;
            scnt[lane + 64] = 0;
        }
    }
    // level bounds, one per lane: lane j holds the start of level j, lane
    // h + 1 the end of the partition (read out by lane index, no memory wait)
    const int32_t spv = A.offs[(int64_t)p * (h + 1) + min(lane, h + 1)];
    const int32_t spn = __shfl_down(spv, 1, 64);   // every lane takes part
    const uint32_t lne = (uint32_t)__builtin_amdgcn_ballot_w64(lane <= h && spv < spn);
    __syncthreads();
#pragma unroll
    for (int i = 0; i < kXW; i++) {
        qa = fmaxf(qa, qmx[0][i]);
        qb = fmaxf(qb, qmx[1][i]);
        lv |= lvw[i];
    }
    // the levels to scan: selected by a query of the tile and not empty
    lv = __builtin_amdgcn_readfirstlane(lv & lne);
    // MFMA B operands: the lane's query, K slice 8g of each step
    uint4 bq[KS];
    {
        const uint8_t *src = A.qlow + (int64_t)my_qq * ROWB + 16 * g;
#pragma unroll
        for (int s = 0; s < KS; s++)
            bq[s] = own ? *reinterpret_cast<const uint4 *>(src + 32 * s) : make_uint4(0u, 0u, 0u, 0u);
    }
    // MFMA A operands: row c32 of a staged chunk, K slice 8g of step s at
    // c32 ROWB + 16 ((2s + g) ^ swizzle) = xo ^ 32s (the row's bytes are a
    // power of two and 2s + g = 2s | g)
    const uint32_t xo = (uint32_t)(c32 * ROWB + 16 * (g ^ ((c32 / RPL) & SWZ)));

    // chunk cursors (wave-uniform): level j, first row c0, end of the level;
    // past the last level j = h + 1
    auto next_level = [&](int &j, int32_t &c0, int32_t &end) {
        const uint32_t rest = lv >> (j + 1);   // j + 1 <= h + 1 <= 16
        if (!rest) {
            j = h + 1;
            return;
        }
        j += 1 + __builtin_ctz(rest);
        c0 = __builtin_amdgcn_readlane(spv, j);
        end = __builtin_amdgcn_readlane(spv, j + 1);
    };
    auto advance1 = [&](int &j, int32_t &c0, int32_t &end) {
        c0 += kXCH;
        if (c0 >= end) next_level(j, c0, end);
    };
    auto advance = [&](int &j, int32_t &c0, int32_t &end) {
        advance1(j, c0, end);
        for (int i = 1; i < nshare; i++) advance1(j, c0, end);
    };

    // Staging.  Every wave issues the same loads per chunk (UPW row loads
    // and one or two per-point loads), always, so that one wait count holds for all
    // waves and every path (a missing chunk loads row 0 into the unused
    // buffer instead).  Row load i, lane L fills tile bytes 1024 i + 16 L:
    // row (64 i + L) / V16, piece (64 i + L) % V16, which holds global piece
    // piece ^ swizzle of the row; rows past the level's end load its last row
    // and are masked by a NaN point term; loads past NDMA (short rows) repeat
    // load i - NDMA.  Per-point load of wave w, lane L: input w (squared
    // norm, error norms, packed dense word) of row c0 + min(L, cn - 1), L < 32;
    // second load: wave 0 the FP8 scales alike, the other waves (or all) the
    // signatures, lane L word L % 2 of row c0 + min(L / 2, cn - 1) (the waves
    // write the same values).
    uint32_t voff[UPW];
    int vrow[UPW];
#pragma unroll
    for (int u = 0; u < UPW; u++) {
        const int i = (w + kXW * u) % NDMA;
        const int slot = 64 * i + lane;
        const int row = slot / V16;
        vrow[u] = row;
        voff[u] = (uint32_t)(row * ROWB + 16 * ((slot % V16) ^ ((row / RPL) & SWZ)));
    }
    constexpr int OPC = UPW + 1 + (PTS2 ? 1 : 0) + (SLOTS ? 1 : 0);   // loads per wave per chunk
    const uint32_t *wsrc = has_dense ? A.words : reinterpret_cast<const uint32_t *>(A.xnorm);
    const float *psrc = w == 0   ? A.xnorm
                        : w == 1 ? A.lerr
                        : w == 2 ? A.lnrm
                                 : reinterpret_cast<const float *>(wsrc);
    // (seed pass with labels: also the slots of rows 8w..8w+7, 16 bytes each;
    // wide rows load the start of the copy in their place)
    auto fetch_rows = [&](bool real, int32_t c0, int cn, uint8_t *dst, uint16_t *sdst) {
        const uint8_t *base = real ? A.lvecs + (int64_t)c0 * ROWB : A.lvecs;
#pragma unroll
        for (int u = 0; u < UPW; u++) {
            const int i = (w + kXW * u) % NDMA;
            uint32_t off = real ? voff[u] : 0u;
            if (real && cn < kXCH) off -= (uint32_t)(max(vrow[u] - (cn - 1), 0) * ROWB);
            __builtin_amdgcn_global_load_lds(base + off, (__attribute__((address_space(3))) void *)(dst + 1024 * i), 16,
                                             0, 0);
        }
        if constexpr (SLOTS) {
            if (lane < 8) {
                const int64_t row = c0 + min(8 * w + lane, cn - 1);
                const void *src = real && narrow ? (const void *)(A.slots + row * kMaxLabels) : (const void *)A.lvecs;
                __builtin_amdgcn_global_load_lds(
                    src, (__attribute__((address_space(3))) void *)(sdst + 8 * w * kMaxLabels), 16, 0, 0);
            }
        }
    };
    auto fetch_points = [&](bool real, int32_t c0, int cn, float (*raw)[kXCH], Raw2 raw2) {
        // lanes 0..31 (lane L fills raw[w][L]; every wave has them active, so
        // the load is issued on every path)
        if (lane < kXCH) {
            const int64_t row = real ? c0 + min(lane, cn - 1) : 0;
            __builtin_amdgcn_global_load_lds(psrc + row, (__attribute__((address_space(3))) void *)raw[w], 4, 0, 0);
        }
        if constexpr (PTS2) {
            // wave-uniform: scales (32 lanes, third array), else signatures
            // (64 lanes, the first two); without labels the FP8 scales from every
            // wave, or (disjunctions without labels) the norms as a stand-in
            if (F8 && (w == 0 || !has_lab)) {
                if (lane < kXCH) {
                    const int64_t row = real ? c0 + min(lane, cn - 1) : 0;
                    __builtin_amdgcn_global_load_lds(A.lscale + row, (__attribute__((address_space(3))) void *)raw2[2], 4,
                                                     0, 0);
                }
            } else {
                const int64_t row = real ? c0 + min(has_lab ? lane >> 1 : lane & 31, cn - 1) : 0;
                const uint32_t *src = has_lab ? reinterpret_cast<const uint32_t *>(A.sigs) + 2 * row + (lane & 1)
                                              : reinterpret_cast<const uint32_t *>(A.xnorm) + row;
                __builtin_amdgcn_global_load_lds(src, (__attribute__((address_space(3))) void *)raw2[0], 4, 0, 0);
            }
        }
    };
    // the point terms of a chunk whose per-point inputs have landed (one
    // wave per chunk, in turn)
    auto point_terms = [&](float (*raw)[kXCH], Raw2 raw2, int cn, int pb) {
        const float nx = raw[0][c32];
        const float slack = fmaf(raw[1][c32], qa, raw[2][c32] * qb) * (1.0f + 0x1p-20f);
        float pt = l2 ? fmaf(-A.eta, nx, fmaf(-2.0f, slack, nx)) : fmaf(-A.eta, nx, -slack);
        if (!(fabsf(pt) < inf)) pt = -inf;
        if (APPROX) pt = l2 ? nx : 0.0f;   // approximate keys: the plain point term
        if constexpr (LAB) {   // (without labels every query's signature, 0, is a subset)
            reinterpret_cast<uint32_t *>(xsig[pb])[lane] = raw2[lane >> 5][c32];
        }
        if constexpr (F8) xsc[pb][c32] = __uint_as_float(raw2[2][c32]);
        xn[pb][c32] = c32 < cn ? pt : qnan;   // (lanes l and l + 32 write alike)
        const uint32_t wd = has_dense ? __float_as_uint(raw[3][c32]) : 0u;
        xw[pb][c32] = wd;
        // the chunk's summary for the skip test: AND and OR of its rows'
        // words, reduced inside each 16-lane row by rotations (DPP row_ror
        // 1, 2, 4, 8), then rows 0 and 1 (lanes 0..31 hold the chunk's rows)
        int wa = c32 < cn ? (int)wd : -1, wo = c32 < cn ? (int)wd : 0;
        wa &= __builtin_amdgcn_mov_dpp(wa, 0x121, 0xF, 0xF, false);
        wo |= __builtin_amdgcn_mov_dpp(wo, 0x121, 0xF, 0xF, false);
        wa &= __builtin_amdgcn_mov_dpp(wa, 0x122, 0xF, 0xF, false);
        wo |= __builtin_amdgcn_mov_dpp(wo, 0x122, 0xF, 0xF, false);
        wa &= __builtin_amdgcn_mov_dpp(wa, 0x124, 0xF, 0xF, false);
        wo |= __builtin_amdgcn_mov_dpp(wo, 0x124, 0xF, 0xF, false);
        wa &= __builtin_amdgcn_mov_dpp(wa, 0x128, 0xF, 0xF, false);
        wo |= __builtin_amdgcn_mov_dpp(wo, 0x128, 0xF, 0xF, false);
        // (the lane reads stay outside the single-lane branch below: they
        // read lanes that branch leaves inactive)
        const uint32_t sa = (uint32_t)(__builtin_amdgcn_readlane(wa, 0) & __builtin_amdgcn_readlane(wa, 16));
        const uint32_t so = (uint32_t)(__builtin_amdgcn_readlane(wo, 0) | __builtin_amdgcn_readlane(wo, 16));
        if (lane == 0) {
            xsum[pb][0] = sa;
            xsum[pb][1] = so;
        }
    };

    // The exact test of a pair's labels: the query's in the point's slots (its
    // dense constraints were tested on the staged words), or each term of a
    // disjunction in full.
    auto rest_passes = [&](int qj, uint32_t pos) -> bool {
        const QDesc &qd = qds[kXQ * w + qj];
        const uint64_t sg = A.sigs[pos];
        const uint16_t *sl = A.slots + (int64_t)pos * A.lslots;
        if (DISJ && (qd.flags & kQOr))
            return query_passes(qd, A.qterms + (int64_t)(ent[kXQ * w + qj] / A.m) * kMaxTerms, has_dense, true,
                                has_dense ? A.words[pos] : 0u, sg, sl, A.lslots);
        return point_passes(qd, false, true, 0u, sg, sl, A.lslots);
    };

    // The test on staged data only: the query's signature bits; for a
    // disjunction some term's dense fields and signature bits.  It leaves
    // rest_passes only the label slots (a disjunction of dense terms nothing).
    const bool any_or = DISJ && __builtin_amdgcn_ballot_w64(my_or) != 0;
    auto staged_passes = [&](uint32_t wd, uint64_t sig) -> bool {
        bool ok = (my_lsig & ~sig) == 0;
        if (any_or) {
            bool some = false;
#pragma unroll
            for (int i = 0; i < (DISJ ? kMaxTerms : 1); i++) some |= (wd & tm[i]) == tv[i] && (tl[i] & ~sig) == 0;
            ok &= some || !my_or;
        }
        return ok;
    };

    // deferred pairs of this wave: (CSR position, wave query) in a ring of
    // 64, appended to their queries' lists when a ballot's pairs would not
    // fit (per-query ranks from an LDS histogram, one returning atomic per
    // query); a query whose list is full is flagged for the rescue pass
    uint32_t *ring_pos = ring[w][0];
    uint32_t *ring_row = ring[w][1];
    uint32_t *ring_key = ring[w][SEED ? 1 : 2];   // the pair's ordered score (not in the seed mode)
    int32_t *hist = dhist[w];
    int vhead = 0, vtail = 0;
    auto drain = [&](int n) {
        wave_sync();
        bool v = lane < n;
        const int slot = (vtail + lane) & (kXRing - 1);
        const uint32_t pos = v ? ring_pos[slot] : 0u;
        const int qj = v ? (int)ring_row[slot] : 0;
        const uint32_t pkey = v ? ring_key[slot] : 0u;
        vtail += n;
        if constexpr (LAB) {
            if (v && has_lab) v = rest_passes(qj, pos);   // (dense terms only: tested)
        }
        if (lane < kXQ) hist[lane] = 0;
        wave_sync();
        const int rank = v ? atomicAdd(hist + qj, 1) : 0;
        wave_sync();
        const int cnt = lane < kXQ ? hist[lane] : 0;
        int base = 0;
        if (cnt > 0) base = atomicAdd(A.dcnt + my_qq, cnt);
        const int at = __shfl(base, qj, 64) + rank;
        const int32_t qq = __shfl(my_qq, qj, 64);
        if (v && at < A.dcap) A.dpos[(int64_t)qq * A.dcap + at] = ((uint64_t)pkey << 32) | pos;
        if (v && at >= A.dcap) A.oflow[qq] = 1;
    };

    // ---- pipeline.  Fetch F_c = rows of chunk c into buffer c % 4 and the
    // per-point inputs of chunk c + 1 into slot (c + 1) % 4.  Step k waits
    // for F_k (two later fetches may stay in flight), passes the barrier,
    // issues F_{k+3}, lets wave k % 4 turn the inputs of chunk k + 1 into its
    // point terms, and scores chunk k.
    int cj = -1;
    int32_t cc0 = 0, cend = 0;
    next_level(cj, cc0, cend);
    for (int i = 0; i < share; i++) advance1(cj, cc0, cend);
    if (cj > h) {   // nothing to scan
        if (SEED && g == 0 && own) {
            if (share == 0) A.pcnt[my_slot] = nshare > 1 ? 2 * MH * nshare : 0;
            if (nshare > 1)
                for (int i = 0; i < 2 * MH; i++) A.partials[(int64_t)my_slot * A.r + share * 2 * MH + i] = ~0ull;
        }
        return;
    }
    // fetch cursor (chunk of the rows of the next fetch) and the chunk after it
    int fj = cj, rj = cj;
    int32_t fc0 = cc0, fend = cend, rc0 = cc0, rend = cend;
    advance(rj, rc0, rend);
    auto fetch_next = [&](uint8_t *dst, uint16_t *sdst, float (*raw)[kXCH], Raw2 raw2) {
        const bool fr = fj <= h, rr = rj <= h;
        fetch_rows(fr, fc0, fr ? min(kXCH, fend - fc0) : 1, dst, sdst);
        fetch_points(rr, rc0, rr ? min(kXCH, rend - rc0) : 1, raw, raw2);
        if (fr) advance(fj, fc0, fend);
        if (rr) advance(rj, rc0, rend);
    };
    fetch_points(true, cc0, min(kXCH, cend - cc0), rw0, rg0);   // the inputs of chunk 0
    fetch_next(xb0, xl0, rw1, rg1);
    fetch_next(xb1, xl1, rw2, rg2);
    fetch_next(xb2, xl2, rw3, rg3);
    // the first three chunks have landed on every wave (waiting for all of
    // them lets the compiler's own wait tracking enter the loop with nothing
    // in flight)
    __builtin_amdgcn_s_waitcnt(0xC07F & 0x0F70);   // vmcnt(0) lgkmcnt(0)
    __builtin_amdgcn_s_barrier();
    if (w == 0) point_terms(rw0, rg0, min(kXCH, cend - cc0), 0);
    int lj = -1;
    float tfj = qnan;
    uint64_t lst[SEED ? MH : 1];   // seed: the lane's best keys, ascending (~0: empty)
#pragma unroll
    for (int i = 0; i < (SEED ? MH : 1); i++) lst[i] = ~0ull;

    // Chunk k from buffer `cur` (point arrays `pb`); `nraw` holds the inputs
    // of chunk k + 1, whose point terms wave `ptw` (k % 4) computes; F_{k+3}
    // goes to `nxt` and `fraw`.  Returns whether another chunk follows.
    auto step = [&](const uint8_t *cur, uint8_t *nxt, const uint16_t *scur, uint16_t *snxt, const int pb, float (*nraw)[kXCH], Raw2 nraw2,
                    float (*fraw)[kXCH], Raw2 fraw2, const int ptw) -> bool {
        const int j = cj;
        const int32_t c0 = cc0;
        const int cn = min(kXCH, cend - c0);
        // F_k has landed once at most the two later fetches are outstanding
        // (stores and atomics issued since only make the wait stricter); the
        // point terms wave 0 wrote are complete
        __builtin_amdgcn_s_waitcnt(0xC07F & (0x0F70 | ((2 * OPC) & 15) | (((2 * OPC) >> 4) << 14)));
        __builtin_amdgcn_s_barrier();
        advance(cj, cc0, cend);
        const bool more = cj <= h;
        fetch_next(nxt, snxt, fraw, fraw2);
        if (w == ptw && more) point_terms(nraw, nraw2, min(kXCH, cend - cc0), pb ^ 1);
        if (kXQ * w >= nqt) return more;   // a wave without queries (small batches) only stages
        {
            // A row passes (w & M) == V only if every bit of V is set in the
            // OR of the chunk's words and every other bit of M is clear in
            // their AND: where no query of the wave can pass a row of the
            // chunk, its products and tests are skipped (the queries of a
            // wave share constraints and a sub-partition's rows are grouped
            // by their values, so this is common)
            const uint32_t wa = xsum[pb][0], wo = xsum[pb][1];
            uint32_t miss = (my_val & ~wo) | (~my_val & my_mask & wa) | (((my_sel >> j) & 1u) ^ 1u);
            if (any_or) {   // a disjunction: some term may pass
                bool some = !my_or;
#pragma unroll
                for (int i = 0; i < (DISJ ? kMaxTerms : 1); i++)
                    some |= ((tv[i] & ~wo) | (~tv[i] & tm[i] & wa)) == 0u;
                if (!some) miss = 1u;
            }
            if (!__builtin_amdgcn_ballot_w64(miss == 0u)) return more;
        }

        f32x16 acc = {};
#pragma unroll
        for (int s0 = 0; s0 < KS; s0 += 2) {   // operands of two steps, then their products
            uint4 a[2];
#pragma unroll
            for (int s = s0; s < s0 + 2 && s < KS; s++) a[s - s0] = *reinterpret_cast<const uint4 *>(cur + (xo ^ (32u * s)));
#pragma unroll
            for (int s = s0; s < s0 + 2 && s < KS; s++) acc = mma32<PREC>(a[s - s0], bq[s], acc);
        }
        if constexpr (F8) {   // both scales
#pragma unroll
            for (int q4 = 0; q4 < 4; q4++) {
                const float4 ps = *reinterpret_cast<const float4 *>(&xsc[pb][8 * q4 + 4 * g]);
                const float sv[4] = {ps.x, ps.y, ps.z, ps.w};
#pragma unroll
                for (int e = 0; e < 4; e++) acc[4 * q4 + e] = acc[4 * q4 + e] * sv[e] * my_qs;
            }
        }

        if constexpr (SEED) {
            // approximate keys below the lane's bound (the shared bound at the
            // tile's start, then the worst of its MH best) that pass the
            // packed dense test enter its sorted list; lanes l and l + 32 keep
            // one list each for query l % 32 (its half of the chunk's points)
            if (j != lj) {
                lj = j;
                tfj = ((my_sel >> j) & 1u) ? bound_score(lst[MH - 1] < my_tk ? lst[MH - 1] : my_tk) : qnan;
            }
            auto offer = [&](uint64_t kk) {   // one compare-exchange pass keeps the list sorted
#pragma unroll
                for (int i = 0; i < MH; i++) {
                    const bool lt = kk < lst[i];
                    const uint64_t lo = lt ? kk : lst[i];
                    kk = lt ? lst[i] : kk;
                    lst[i] = lo;
                }
                tfj = bound_score(lst[MH - 1] < my_tk ? lst[MH - 1] : my_tk);
            };
            uint32_t cand = 0;   // label variant: elements that passed the score, dense and signature tests
#pragma unroll
            for (int q4 = 0; q4 < 4; q4++) {
                const int rb = 8 * q4 + 4 * g;
                const float4 pn = *reinterpret_cast<const float4 *>(&xn[pb][rb]);
                const float pv[4] = {pn.x, pn.y, pn.z, pn.w};
                uint64_t hit[4];
#pragma unroll
                for (int e = 0; e < 4; e++) {
                    acc[4 * q4 + e] = fmaf(cm, acc[4 * q4 + e], pv[e]);
                    hit[e] = __builtin_amdgcn_ballot_w64(acc[4 * q4 + e] <= tfj);
                }
                if (!(hit[0] | hit[1] | hit[2] | hit[3])) continue;
                const uint4 pw = *reinterpret_cast<const uint4 *>(&xw[pb][rb]);
                const uint32_t wv[4] = {pw.x, pw.y, pw.z, pw.w};
#pragma unroll
                for (int e = 0; e < 4; e++) {
                    if (!((hit[e] >> lane) & 1ull) || (wv[e] & my_mask) != my_val) continue;
                    if constexpr (LAB) {
                        if (staged_passes(wv[e], !DISJ || has_lab ? xsig[pb][rb + e] : ~0ull)) cand |= 1u << (4 * q4 + e);
                    } else {
                        const uint64_t key = ((uint64_t)f2ord(canon0(acc[4 * q4 + e])) << 32) | (uint32_t)(c0 + rb + e);
                        if (key < lst[MH - 1]) offer(key);
                    }
                }
            }
            if constexpr (LAB) {   // their labels (or terms), in one copy of the code
                while (cand) {
                    const int r = __builtin_ctz(cand);
                    cand &= cand - 1u;
                    float sc = acc[0];
#pragma unroll
                    for (int e = 1; e < 16; e++) sc = r == e ? acc[e] : sc;
                    const uint32_t pos = (uint32_t)(c0 + 8 * (r >> 2) + 4 * g + (r & 3));
                    const uint64_t key = ((uint64_t)f2ord(canon0(sc)) << 32) | pos;
                    if (!(key < lst[MH - 1])) continue;
                    bool ok;
                    if (!has_lab) {
                        ok = true;   // (dense terms only: tested)
                    } else if (narrow && !my_or) {   // the labels against the staged slots
                        const uint16_t *sl = scur + (pos - c0) * kMaxLabels;
                        const QDesc &qd = qds[kXQ * w + c32];
                        ok = true;
                        for (int i = 0; i < qd.nlab; i++) ok &= slots_hold(sl, kMaxLabels, qd.lab[i]);
                    } else {
                        ok = rest_passes(c32, pos);
                    }
                    if (ok) offer(key);
                }
            }
        } else {
            if (j != lj) {   // level changed: the query's bound if it selects the level, NaN if not
                lj = j;
                tfj = ((my_sel >> j) & 1u) ? my_tf : qnan;
            }
            const bool sj = (my_sel >> j) & 1u;
            // point terms of the next group read while this one is scored
            float4 pnx = *reinterpret_cast<const float4 *>(&xn[pb][4 * g]);
#pragma unroll
            for (int q4 = 0; q4 < 4; q4++) {   // points 8 q4 + 4 g + e of the chunk, e < 4
                const int rb = 8 * q4 + 4 * g;
                const float4 pn = pnx;
                if (q4 < 3) pnx = *reinterpret_cast<const float4 *>(&xn[pb][rb + 8]);
                const float pv[4] = {pn.x, pn.y, pn.z, pn.w};
                uint64_t hit[4];
                float sc[4];   // the element test's scores (deferred with their pairs)
#pragma unroll
                for (int e = 0; e < 4; e++) {
                    sc[e] = fmaf(cm, acc[4 * q4 + e], pv[e]);
                    hit[e] = __builtin_amdgcn_ballot_w64(sc[e] <= tfj);
                }
                if constexpr (COUNT) {   // survivors of the exact filter (statistics only)
                    const uint4 pw = *reinterpret_cast<const uint4 *>(&xw[pb][rb]);
                    const uint32_t wv[4] = {pw.x, pw.y, pw.z, pw.w};
                    int c = 0;
#pragma unroll
                    for (int e = 0; e < 4; e++) c += (sj && rb + e < cn && (wv[e] & my_mask) == my_val) ? 1 : 0;
                    if (c) atomicAdd(&scnt[qi], c);
                }
                if (!(hit[0] | hit[1] | hit[2] | hit[3])) continue;
                {   // the packed dense test where a score passed
                    const uint4 pw = *reinterpret_cast<const uint4 *>(&xw[pb][rb]);
                    const uint32_t wv[4] = {pw.x, pw.y, pw.z, pw.w};
#pragma unroll
                    for (int e = 0; e < 4; e++) hit[e] &= __builtin_amdgcn_ballot_w64((wv[e] & my_mask) == my_val);
                    if constexpr (LAB) {   // then the label signatures
                        if (!(hit[0] | hit[1] | hit[2] | hit[3])) continue;
#pragma unroll
                        for (int e = 0; e < 4; e++)
                            hit[e] &= __builtin_amdgcn_ballot_w64(
                                staged_passes(wv[e], !DISJ || has_lab ? xsig[pb][rb + e] : ~0ull));
                    }
                }
#pragma unroll
                for (int e = 0; e < 4; e++) {
                    const uint64_t hm = hit[e];
                    if (!hm) continue;
                    const int n = __popcll(hm);   // at most 64
                    if (vhead - vtail + n > kXRing) drain(vhead - vtail);
                    if ((hm >> lane) & 1ull) {
                        const int sl = (vhead + __popcll(hm & lanemask_lt())) & (kXRing - 1);
                        ring_pos[sl] = (uint32_t)(c0 + rb + e);
                        ring_row[sl] = (uint32_t)c32;
                        ring_key[sl] = f2ord(canon0(sc[e]));
                    }
                    vhead += n;
                }
            }
        }
        return more;
    };
    while (step(xb0, xb3, xl0, xl3, 0, rw1, rg1, rw0, rg0, 0) && step(xb1, xb0, xl1, xl0, 1, rw2, rg2, rw1, rg1, 1) &&
           step(xb2, xb1, xl2, xl1, 0, rw3, rg3, rw2, rg2, 2) && step(xb3, xb2, xl3, xl2, 1, rw0, rg0, rw3, rg3, 3)) {
    }
    if constexpr (SEED) {
        // the slot's list: the keys of half 0, then those of half 1 (2 MH <= r
        // entries); a full list of r keys bounds the query's r-th key
        int cnt = 0;
#pragma unroll
        for (int i = 0; i < MH; i++) cnt += lst[i] != ~0ull ? 1 : 0;
        const int c_lo = __shfl(cnt, c32, 64);
        const int c_hi = __shfl(cnt, c32 + 32, 64);
        const uint64_t w_hi = ((uint64_t)(uint32_t)__shfl((int)(lst[MH - 1] >> 32), c32 + 32, 64) << 32) |
                              (uint32_t)__shfl((int)(uint32_t)lst[MH - 1], c32 + 32, 64);
        if (own && nshare > 1) {   // each share fills its part of the list (2 MH nshare <= r), padding included
            uint64_t *out = A.partials + (int64_t)my_slot * A.r + share * 2 * MH + g * MH;
#pragma unroll
            for (int i = 0; i < MH; i++) out[i] = lst[i];
            if (g == 0 && share == 0) A.pcnt[my_slot] = 2 * MH * nshare;
        } else if (own) {
            uint64_t *out = A.partials + (int64_t)my_slot * A.r + (g ? c_lo : 0);
#pragma unroll
            for (int i = 0; i < MH; i++)
                if (i < cnt) out[i] = lst[i];
            if (g == 0) {
                A.pcnt[my_slot] = c_lo + c_hi;
                if (c_lo + c_hi == A.r) {
                    const uint64_t worst = lst[MH - 1] > w_hi ? lst[MH - 1] : w_hi;
                    // (one past it: the main pass covers this probe again)
                    atomicMin((unsigned long long *)(A.tau + my_qq), (unsigned long long)worst + 1ull);
                }
            }
        }
        return;
    } else {
        if (vhead > vtail) drain(vhead - vtail);
        if constexpr (COUNT) {
            __syncthreads();
            if (g == 0 && own && scnt[qi]) atomicAdd(&A.nsurv[my_qq], scnt[qi]);
        }
    }
}

// The kernel for rows of ns 32-element steps (ns <= 4; caps_x32_inst.hip) and a
// filter kind (0 dense values, 1 labels too, 2 disjunctions too): mode 0 exact
// main pass, 1 counting survivors (filter kind 0 only), 2 seed lists of one
// key, 3 of four keys per half of a partition's rows, 4 approximate main pass.
template <int PREC, int FILT>
LowpFn pick_x32(int ns, int mode);
#define CAPS_X32_DECL(P)                              \
    template <> LowpFn pick_x32<P, 0>(int, int);      \
    template <> LowpFn pick_x32<P, 1>(int, int);      \
    template <> LowpFn pick_x32<P, 2>(int, int);
CAPS_X32_DECL(CAPS_PREC_BF16)
CAPS_X32_DECL(CAPS_PREC_FP16)
CAPS_X32_DECL(CAPS_PREC_FP8)
#undef CAPS_X32_DECL

}  // namespace caps
