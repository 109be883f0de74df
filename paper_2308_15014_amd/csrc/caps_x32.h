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
//  * rows come in chunks of 32, two chunks a step, staged by direct loads one
//    step ahead into two buffers; one barrier a step.  Which rows a chunk holds
//    is laid out for 64 chunks at once, one per lane, and read out by lane
//    index (a cursor advanced per chunk cost 100 scalar instructions a chunk);
//  * a chunk is skipped where the AND and OR of its rows' packed words show
//    that no query of the wave passes, without labels also where no row passes
//    any query's packed test;
//  * the filter test of an element runs on staged words: the packed dense
//    fields and, in the bits they leave free, the label signature folded, in
//    one masked compare; then the signature.  The main pass makes the rest
//    (label slots, terms of disjunctions; global reads) when it drains a wave's
//    ring of pairs, one pair per lane, so that one round trip to memory serves
//    up to 64 pairs.
// What bounds it: the chain of waits of a step, with four waves per SIMD (BF16
// main pass: matrix cores busy 14 % of the time, vector units about 60 %, 54 %
// of the wave time waiting).  Before the steps of two
// chunks, the masks of passing elements (instead of branches per element) and
// the folded signatures: main pass of 10k queries x 1M x 128 BF16 1.73 ms, now
// 1.63; 4k queries, labels, 96-d FP8 3.16, now 2.46; 8k queries, dense values
// and labels, 2M FP16 5.59, now 4.98; their seed passes 0.25, 0.70 and 1.37 ms,
// now 0.23, 0.46 and 1.04.  Two blocks of queries per wave (half the steps, but
// 3 and 2 waves per SIMD) ran 1.83, 4.40 and 7.86 ms.
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
// bound's margin covers for any order.  Approximate scores are results of
// their own (which candidates are rescored, and ties among them, follow from
// their rounding), so those modes exchange halves between the lanes of a pair
// first (fp8_ascend): the products then sum ascending elements, bit for bit as
// k_scan_mfma's 16 x 16 x 32 products do.  (So do the two-byte formats'.)
#pragma once

#include "caps_mfma.h"

namespace caps {

constexpr int kXG = 2;                 // chunks per step
constexpr int kXW = 2 * kXG;           // waves per tile
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

// Lane l holds bytes 16 g.. of a row's 32-byte block (g = l / 32); afterwards
// its first half holds bytes 8 g.. and its second half bytes 16 + 8 g.., the
// operands of two products over ascending elements.
__device__ inline uint4 fp8_ascend(uint4 v) {
    const auto lo = __builtin_amdgcn_permlane32_swap(v.x, v.z, false, false);
    const auto hi = __builtin_amdgcn_permlane32_swap(v.y, v.w, false, false);
    return make_uint4(lo[0], hi[0], lo[1], hi[1]);
}

// A label signature folded into the bits of the packed word that no dense field
// uses (nfree of them from bit `at` on): the query's folded bits are a subset
// of those of every point that holds its labels, so the one masked compare of
// the packed words refuses most pairs that fail the labels.  nfree 0: no bits.
__device__ inline uint32_t fold_sig(uint64_t sig, int at, int nfree) {
    if (nfree == 0) return 0u;
    uint64_t f = 0;
    for (int s = 0; s < 64; s += nfree) f |= sig >> s;
    return (uint32_t)(f & ((1ull << nfree) - 1ull)) << at;
}

// Waves per SIMD the registers are budgeted for.  A step is a chain of waits
// (LDS operands, products, tests), so a fourth wave beats the registers it
// costs: FP8 labels 2.46 against 3.04 ms in the main pass and 0.56 against
// 0.65 ms in the seed pass although 22 registers spill there, FP16 labels 5.03
// against 5.47 ms.  Disjunctions (their terms in registers), seed lists of
// four keys with labels and the counting pass (12 registers would spill) stay
// at three; so, by its LDS (41,120 bytes: the staged label slots), does the
// seed pass with labels on two-byte rows of 128 elements.  FP8 has the registers
// for a fourth wave of the counting pass, and for a fifth of the main pass on
// rows of 32 elements (two spill; with four waves 137 us against 119 for 1320
// queries over 195 of 545 partitions).
constexpr int x32_waves(int prec, int ns, int mode, int mh, int filt) {
    if (prec == CAPS_PREC_FP8 && filt == 0 && mode == 1) return 4;
    if (prec == CAPS_PREC_FP8 && filt == 0 && mode == 0 && ns == 1) return 5;
    return filt == 2 || mode == 1 || (filt == 1 && mode == 2 && mh > 1) ? 3 : 4;
}

template <int PREC, int NS, int MODE, int MH, int FILT>
__global__ __launch_bounds__(kXW * 64) __attribute__((amdgpu_waves_per_eu(x32_waves(PREC, NS, MODE, MH, FILT)))) void k_scan_x32(LowpArgs A) {
    constexpr bool LAB = FILT != 0;     // label tests (an index with labels)
    constexpr bool DISJ = FILT == 2;    // and disjunctions, on any index
    static_assert(!(LAB && MODE == 1), "survivors of label tests are counted by k_scan_mfma");
    constexpr bool COUNT = MODE == 1;   // survivor counts of the exact filter
    constexpr bool SEED = MODE == 2;    // approximate keys: per query and probe the best 2 MH
    constexpr bool APPROX = MODE >= 2;  // approximate scores (no margin)
    constexpr bool F8 = PREC == CAPS_PREC_FP8;
    constexpr int ROWB = NS * (F8 ? 32 : 64);      // bytes per row of the copy
    constexpr int KS = ROWB / 32;                  // 16-byte operands per lane and row
    constexpr int V16 = ROWB / 16;                 // 16-byte pieces per row
    constexpr int NDMA = kXCH * ROWB / 1024;       // 1 KB direct loads per chunk
    constexpr int UPW = (kXG * NDMA + kXW - 1) / kXW;
    constexpr int RPL = ROWB >= 256 ? 1 : 256 / ROWB;
    constexpr int SWZ = ROWB >= 256 ? 15 : V16 - 1;
    constexpr int PRE = APPROX ? 2 : 4;            // per-point inputs per row (approximate scores: no error norms)
    constexpr int GR = kXG * kXCH;                 // rows per step
    // the two row buffers: distinct arrays, so that the compiler can tell
    // the reads of one from the direct loads into the other
    __shared__ __align__(16) uint8_t xb0[GR * ROWB];
    __shared__ __align__(16) uint8_t xb1[GR * ROWB];
    __shared__ __align__(16) float rw0[PRE][GR];   // the per-point inputs of each buffer's rows
    __shared__ __align__(16) float rw1[PRE][GR];
    // label signatures (two words each), FP8 scales
    __shared__ __align__(16) uint32_t rg0[LAB ? 2 * GR : 1];
    __shared__ __align__(16) uint32_t rg1[LAB ? 2 * GR : 1];
    __shared__ __align__(16) float rs0[F8 ? GR : 1];
    __shared__ __align__(16) float rs1[F8 ? GR : 1];
    __shared__ __align__(16) uint64_t xsig[LAB ? 2 : 1][LAB ? GR : 1];   // signatures of the scored rows
    __shared__ __align__(16) float xsc[F8 ? 2 : 1][F8 ? GR : 1];         // FP8 scales of the scored rows
    // seed pass: the label slots of narrow rows (8 of them), beside the rows of each buffer
    constexpr bool SLOTS = SEED && LAB;
    __shared__ __align__(16) uint16_t xl0[SLOTS ? GR * kMaxLabels : 1];
    __shared__ __align__(16) uint16_t xl1[SLOTS ? GR * kMaxLabels : 1];
    __shared__ __align__(16) uint4 qlab[SLOTS ? kXQB : 1];   // the tile's query labels (8 of 16 bits)
    __shared__ __align__(16) uint32_t xw[2][GR];
    __shared__ __align__(16) float xn[2][GR];
    __shared__ uint32_t xsum[2][kXG][2];   // AND and OR of each point slot's packed words (the chunk's rows)
    __shared__ uint32_t ring[SEED ? 1 : kXW][2][SEED ? 1 : kXRing];
    __shared__ uint8_t rrow[SEED ? 1 : kXW][SEED ? 1 : kXRing];
    __shared__ int32_t dhist[SEED ? 1 : kXW][kXQ];   // (before the pipeline starts: also the tile's maxima, below)
    __shared__ int32_t scnt[COUNT ? kXQB : 1];   // (only the counting mode: the main passes keep 4 workgroups per CU)
    // the tile prologue's per-wave maxima share the drain histograms' storage:
    // every read of them completes before the pipeline's first barrier, and
    // no drain runs before it
    static_assert(3 * kXW <= kXQ, "the maxima fit in one wave's histogram");
    float(*qmx)[kXW] = reinterpret_cast<float(*)[kXW]>(&dhist[0][0]);
    uint32_t *lvw = reinterpret_cast<uint32_t *>(&dhist[0][2 * kXW]);

    const int slot_i = xcd_tile(blockIdx.x, A.ntiles * A.split);
    if (slot_i < 0) return;
    // the workgroup's share of the tile's rows: chunks share, share + nshare, ...
    // (one of A.split, or what a small batch's tile names; a whole tile has w = 0)
    int tile = slot_i, share = 0, nshare = 1;
    if (A.split > 1) {
        nshare = A.split;
        tile = slot_i / nshare;
        share = slot_i - tile * nshare;
    }
    const int4 dsc = A.tiles[tile];
    if (dsc.w) {
        share = dsc.w & 255;
        nshare = dsc.w >> 8;
    }
    if (dsc.z <= 0) return;
    const int p = dsc.x;
    const int nqt = dsc.z;
    const int32_t *ent = A.entries + dsc.y;
    const int h = A.h;
    const int t = threadIdx.x, lane = t & 63;
    const int w = __builtin_amdgcn_readfirstlane(t >> 6);   // (wave-uniform: kept in a scalar register)
    const int g = lane >> 5, c32 = lane & 31;
    const bool has_dense = A.words != nullptr;
    const bool has_lab = LAB && A.sigs != nullptr;
    const bool narrow = SLOTS && has_lab && A.lslots == kMaxLabels;
    const int nfree = has_lab && A.wbits <= 24 ? 32 - A.wbits : 0;   // (fewer than 8 bits refuse little)
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
    int32_t my_nlab = 0;      // seed: the query's label constraints
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
            const uint32_t fold = fold_sig(qd.lsig, A.wbits, nfree);
            my_mask = qd.dmask | fold;
            my_val = qd.dval | fold;
            my_lsig = qd.lsig;
            my_or = DISJ && (qd.flags & kQOr) != 0;
            if constexpr (SLOTS) {
                my_nlab = qd.nlab;
                const uint16_t *l = qd.lab;   // (read by this wave only)
                if (g == 0)
                    qlab[qi] = make_uint4(l[0] | (uint32_t)l[1] << 16, l[2] | (uint32_t)l[3] << 16,
                                          l[4] | (uint32_t)l[5] << 16, l[6] | (uint32_t)l[7] << 16);
            }
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
        if (w < kXQB / 64) scnt[t] = 0;
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
        if constexpr (F8 && APPROX) {
#pragma unroll
            for (int s = 0; s < KS; s++) bq[s] = fp8_ascend(bq[s]);
        }
    }
    // MFMA A operands: row c32 of a staged chunk, K slice 8g of step s at
    // c32 ROWB + 16 ((2s + g) ^ swizzle) = xo ^ 32s (the row's bytes are a
    // power of two and 2s + g = 2s | g)
    const uint32_t xo = (uint32_t)(c32 * ROWB + 16 * (g ^ ((c32 / RPL) & SWZ)));

    // The tile's chunks: each selected level in steps of kXCH rows, numbered
    // through; with several shares this one's are share, share + nshare, ...
    // Lane L keeps chunk cb + L (first row; level | rows << 8, or 0 past the
    // last), laid out 64 at a time by all lanes at once: a step reads its
    // chunks out by lane index and runs no cursor of its own.
    int32_t ccnt = lane <= h && ((lv >> lane) & 1u) ? (spn - spv + kXCH - 1) / kXCH : 0;
    const int32_t ccum = wave_incl_scan(ccnt);
    int cb = 0;
    int32_t vc0 = 0;
    uint32_t vjc = 0;
    auto plan = [&](int base) {
        cb = base;
        const int x = share + nshare * (base + lane);
        int j = 0;
        for (int e = 0; e <= h; e++) j += __builtin_amdgcn_readlane(ccum, e) <= x ? 1 : 0;
        const int jj = min(j, h);
        const int c0 = __shfl(spv, jj, 64) + kXCH * (x - __shfl(ccum - ccnt, jj, 64));
        const int end = __shfl(spn, jj, 64);
        vc0 = c0;
        vjc = j <= h ? (uint32_t)(j | min(kXCH, end - c0) << 8) : 0u;
    };
    auto chunk0 = [&](int x) -> int32_t { return __builtin_amdgcn_readlane(vc0, x - cb); };
    auto chunkj = [&](int x) -> uint32_t { return __builtin_amdgcn_readlane(vjc, x - cb); };

    // Staging of a step's kXG chunks.  Row load i (1 KB), lane L fills bytes
    // 1024 i + 16 L of the buffer: row (64 i + L) / V16, piece (64 i + L) %
    // V16, which holds global piece piece ^ swizzle of the row; rows past the
    // level's end load its last row and are masked by a NaN point term.
    uint32_t voff[UPW];
    int vrow[UPW];
#pragma unroll
    for (int u = 0; u < UPW; u++) {
        const int slot = 64 * ((w + kXW * u) % NDMA) + lane;
        const int row = slot / V16;
        vrow[u] = row;
        voff[u] = (uint32_t)(row * ROWB + 16 * ((slot % V16) ^ ((row / RPL) & SWZ)));
    }
    // per-point loads: wave w input w % 4 (squared norm, error norms, packed
    // dense word) of the chunks 2 (w / 4) and 2 (w / 4) + 1, 32 lanes each;
    // the FP8 scales alike by the waves from kXG on, the signatures of chunk w
    // by the first kXG waves, lane L word L % 2 of row L / 2
    const uint32_t *wsrc = has_dense ? A.words : reinterpret_cast<const uint32_t *>(A.xnorm);
    const float *psrc = (w & 3) == 0   ? A.xnorm
                        : (w & 3) == 1 ? A.lerr
                        : (w & 3) == 2 ? A.lnrm
                                       : reinterpret_cast<const float *>(wsrc);
    auto fetch_rows = [&](int x, uint8_t *dst, uint16_t *sdst) {   // of chunks x, x + 1, ...
#pragma unroll
        for (int u = 0; u < UPW; u++) {
            const int i = w + kXW * u;
            if (i >= kXG * NDMA) break;
            const uint32_t jc = chunkj(x + i / NDMA);
            if (!jc) break;
            const int cn = (int)(jc >> 8);
            uint32_t off = voff[u];
            if (cn < kXCH) off -= (uint32_t)(max(vrow[u] - (cn - 1), 0) * ROWB);
            __builtin_amdgcn_global_load_lds(A.lvecs + (int64_t)chunk0(x + i / NDMA) * ROWB + off,
                                             (__attribute__((address_space(3))) void *)(dst + 1024 * i), 16, 0, 0);
        }
        if constexpr (SLOTS) {   // the label slots of narrow rows: 16 rows a wave, 16 bytes each
            const uint32_t jc = chunkj(x + w / 2);
            if (narrow && jc && lane < 16) {
                const int64_t row = chunk0(x + w / 2) + min(16 * (w & 1) + lane, (int)(jc >> 8) - 1);
                __builtin_amdgcn_global_load_lds(A.slots + row * kMaxLabels,
                                                 (__attribute__((address_space(3))) void *)(sdst + 16 * w * kMaxLabels),
                                                 16, 0, 0);
            }
        }
    };
    auto fetch_points = [&](int x, float (*raw)[GR], uint32_t *rsig, float *rsc) {
        const bool scales = F8 && w >= kXG && w < kXG + kXG / 2;
        // lane L: row L % 32 of chunk x + 2 (w / 4) + L / 32 (the first one's again if there is no second)
        auto pair_row = [&](int c) -> int64_t {
            const uint32_t ja = chunkj(c), jb = chunkj(c + 1);
            const int32_t ra = chunk0(c) + min(c32, (int)(ja >> 8) - 1);
            const int32_t rb = chunk0(c + 1) + min(c32, (int)(jb >> 8) - 1);
            return g && jb ? rb : ra;
        };
        const int c = x + 2 * (w >> 2);
        const int in = w & 3;
        if ((!APPROX || in == 0 || in == 3) && chunkj(c))
            __builtin_amdgcn_global_load_lds(psrc + pair_row(c),
                                             (__attribute__((address_space(3))) void *)(raw[min(in, PRE - 1)] + 2 * kXCH * (w >> 2)),
                                             4, 0, 0);
        if (scales && chunkj(x + 2 * (w - kXG)))
            __builtin_amdgcn_global_load_lds(A.lscale + pair_row(x + 2 * (w - kXG)),
                                             (__attribute__((address_space(3))) void *)(rsc + 2 * kXCH * (w - kXG)), 4, 0, 0);
        if (LAB && has_lab && w < kXG) {
            const uint32_t jc = chunkj(x + w);
            if (jc) {
                const int64_t row = chunk0(x + w) + min(lane >> 1, (int)(jc >> 8) - 1);
                __builtin_amdgcn_global_load_lds(reinterpret_cast<const uint32_t *>(A.sigs) + 2 * row + (lane & 1),
                                                 (__attribute__((address_space(3))) void *)(rsig + 2 * kXCH * w), 4, 0, 0);
            }
        }
    };
    // the point terms of chunk ci of a step whose per-point inputs have landed
    // (one wave per chunk)
    auto point_terms = [&](float (*raw)[GR], const uint32_t *rsig, const float *rsc, const int ci, int cn, int pb) {
        const int at = kXCH * ci + c32;
        const float nx = raw[0][at];
        float pt = l2 ? nx : 0.0f;   // approximate keys: the plain point term
        if constexpr (!APPROX) {
            const float slack = fmaf(raw[1][at], qa, raw[2][at] * qb) * (1.0f + 0x1p-20f);
            pt = l2 ? fmaf(-A.eta, nx, fmaf(-2.0f, slack, nx)) : fmaf(-A.eta, nx, -slack);
            if (!(fabsf(pt) < inf)) pt = -inf;
        }
        if constexpr (LAB) {   // (without labels every query's signature, 0, is a subset)
            reinterpret_cast<uint32_t *>(xsig[pb])[2 * kXCH * ci + lane] = rsig[2 * kXCH * ci + lane];
        }
        if constexpr (F8) xsc[pb][at] = rsc[at];
        xn[pb][at] = c32 < cn ? pt : qnan;   // (lanes l and l + 32 write alike)
        uint32_t wd = has_dense ? __float_as_uint(raw[PRE - 1][at]) : 0u;
        if constexpr (LAB) wd |= fold_sig(((const uint64_t *)rsig)[at], A.wbits, nfree);
        xw[pb][at] = wd;
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
            xsum[pb][ci][0] = sa;
            xsum[pb][ci][1] = so;
        }
    };

    // The exact test of a pair's labels: the query's in the point's slots (its
    // dense constraints were tested on the staged words), or each term of a
    // disjunction in full.
    auto rest_passes = [&](int32_t qq, uint32_t pos) -> bool {
        const QDesc &qd = A.qd[qq];
        const uint64_t sg = A.sigs[pos];
        const uint16_t *sl = A.slots + (int64_t)pos * A.lslots;
        if (DISJ && (qd.flags & kQOr))
            return query_passes(qd, A.qterms + (int64_t)qq * kMaxTerms, has_dense, true,
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
    uint32_t *ring_pos = ring[SEED ? 0 : w][0];
    uint8_t *ring_row = rrow[SEED ? 0 : w];
    uint32_t *ring_key = ring[SEED ? 0 : w][1];   // the pair's ordered score (not in the seed mode)
    int32_t *hist = dhist[SEED ? 0 : w];
    int vhead = 0, vtail = 0;
    int lj = -1;        // level of the last scored chunk, and the lane's bound there
    float tfj = qnan;
    auto drain = [&](int n) {
        wave_sync();
        bool v = lane < n;
        const int slot = (vtail + lane) & (kXRing - 1);
        const uint32_t pos = v ? ring_pos[slot] : 0u;
        const int qj = v ? (int)ring_row[slot] : 0;
        const uint32_t pkey = v ? ring_key[slot] : 0u;
        vtail += n;
        const int32_t qq = __shfl(my_qq, qj, 64);
        if constexpr (LAB) {
            if (v && has_lab) v = rest_passes(qq, pos);   // (dense terms only: tested)
        }
        if (lane < kXQ) hist[lane] = 0;
        wave_sync();
        const int rank = v ? atomicAdd(hist + qj, 1) : 0;
        wave_sync();
        const int cnt = lane < kXQ ? hist[lane] : 0;
        int base = 0;
        if (cnt > 0) base = atomicAdd(A.dcnt + my_qq, cnt);
        const int at = __shfl(base, qj, 64) + rank;
        if (v && at < A.dcap) A.dpos[(int64_t)qq * A.dcap + at] = ((uint64_t)pkey << 32) | pos;
        if (v && at >= A.dcap) A.oflow[qq] = 1;
        if constexpr (F8) {
            // a query whose list is full is rescanned: no more pairs of it (a
            // round trip to its counter for every 64 of them: 1.72 ms against
            // 0.39 for 2141 queries of which each has 6000).  The two-byte
            // formats' bounds leave few such queries, and the two registers
            // this takes cost their main pass 2 %.
            const uint64_t full = __builtin_amdgcn_ballot_w64(cnt > 0 && base + cnt > A.dcap);
            if ((full >> c32) & 1ull) my_tf = tfj = qnan;
        }
    };

    // ---- pipeline.  Step k scores group k (kXG chunks): it waits for the
    // group's rows (fetched during step k - 1), passes the barrier, fetches the
    // rows of group k + 1 and the per-point inputs of group k + 2 and has one
    // wave per chunk turn the inputs of group k + 1 into point terms.
    plan(0);
    if (!chunkj(0)) {   // nothing to scan
        if (SEED && g == 0 && own) {
            if (share == 0) A.pcnt[my_slot] = nshare > 1 ? 2 * MH * nshare : 0;
            if (nshare > 1)
                for (int i = 0; i < 2 * MH; i++) A.partials[(int64_t)my_slot * A.r + share * 2 * MH + i] = ~0ull;
        }
        return;
    }
    int x = 0;   // first chunk of the scored group
    fetch_points(0, rw0, rg0, rs0);
    fetch_rows(0, xb0, xl0);
    fetch_points(kXG, rw1, rg1, rs1);
    // (waiting for all of them lets the compiler's own wait tracking enter the
    // loop with nothing in flight)
    __builtin_amdgcn_s_waitcnt(0x0F70);   // vmcnt(0)
    lds_barrier();
    if (w < kXG && chunkj(w)) point_terms(rw0, rg0, rs0, w, (int)(chunkj(w) >> 8), 0);
    uint64_t lst[SEED ? MH : 1];   // seed: the lane's best keys, ascending (~0: empty)
#pragma unroll
    for (int i = 0; i < (SEED ? MH : 1); i++) lst[i] = ~0ull;

    // One chunk (ci of group buffer `pb`): its products and tests.
    auto score = [&](const uint8_t *cur, const uint16_t *scur, const int pb, const int ci, const int32_t c0, const int j,
                     const int cn) {
        cur += ci * kXCH * ROWB;
        const int rb0 = ci * kXCH;
        {
            // A row passes (w & M) == V only if every bit of V is set in the
            // OR of the chunk's words and every other bit of M is clear in
            // their AND: where no query of the wave can pass a row of the
            // chunk, its products and tests are skipped (the queries of a
            // wave share constraints and a sub-partition's rows are grouped
            // by their values, so this is common)
            const uint32_t wa = xsum[pb][ci][0], wo = xsum[pb][ci][1];
            uint32_t miss = (my_val & ~wo) | (~my_val & my_mask & wa) | (((my_sel >> j) & 1u) ^ 1u);
            if (any_or) {   // a disjunction: some term may pass
                bool some = !my_or;
#pragma unroll
                for (int i = 0; i < (DISJ ? kMaxTerms : 1); i++)
                    some |= ((tv[i] & ~wo) | (~tv[i] & tm[i] & wa)) == 0u;
                if (!some) miss = 1u;
            }
            if (!__builtin_amdgcn_ballot_w64(miss == 0u)) return;
            if constexpr (!LAB) {
                // then each row against each query, still before the products:
                // the least difference is 0 where a row passes.  (With labels
                // too few blocks go without a pass: 2.60 against 2.42 ms.)
                uint32_t diff = ~0u;
                int cnt = 0;   // survivors of the exact filter (the counting mode)
#pragma unroll
                for (int q4 = 0; q4 < 4; q4++) {
                    const uint4 pw = *reinterpret_cast<const uint4 *>(&xw[pb][rb0 + 8 * q4 + 4 * g]);
                    const uint32_t wv[4] = {pw.x, pw.y, pw.z, pw.w};
#pragma unroll
                    for (int e = 0; e < 4; e++) {
                        const uint32_t x = (wv[e] & my_mask) ^ my_val;
                        diff = min(diff, x);
                        if (COUNT) cnt += 8 * q4 + 4 * g + e < cn && x == 0u ? 1 : 0;
                    }
                }
                if (!__builtin_amdgcn_ballot_w64((miss | diff) == 0u)) return;
                if (COUNT && ((my_sel >> j) & 1u) && cnt) atomicAdd(&scnt[qi], cnt);
                // (the words are read again below: kept in registers across
                // the products they spilled others, 2.49 ms against 1.61)
                wave_sync();
            }
        }

        f32x16 acc = {};
#pragma unroll
        for (int s0 = 0; s0 < KS; s0 += 2) {   // operands of two steps, then their products
            uint4 a[2];
#pragma unroll
            for (int s = s0; s < s0 + 2 && s < KS; s++) a[s - s0] = *reinterpret_cast<const uint4 *>(cur + (xo ^ (32u * s)));
#pragma unroll
            for (int s = s0; s < s0 + 2 && s < KS; s++)
                acc = mma32<PREC>(F8 && APPROX ? fp8_ascend(a[s - s0]) : a[s - s0], bq[s], acc);
        }
        if constexpr (F8) {   // both scales
#pragma unroll
            for (int q4 = 0; q4 < 4; q4++) {
                const float4 ps = *reinterpret_cast<const float4 *>(&xsc[pb][rb0 + 8 * q4 + 4 * g]);
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
            if constexpr (!LAB && MH > 1) {   // several keys a lane: element by element
#pragma unroll
                for (int q4 = 0; q4 < 4; q4++) {
                    const int rb = 8 * q4 + 4 * g;
                    const float4 pn = *reinterpret_cast<const float4 *>(&xn[pb][rb0 + rb]);
                    const float pv[4] = {pn.x, pn.y, pn.z, pn.w};
                    uint64_t hit[4];
#pragma unroll
                    for (int e = 0; e < 4; e++) {
                        acc[4 * q4 + e] = fmaf(cm, acc[4 * q4 + e], pv[e]);
                        hit[e] = __builtin_amdgcn_ballot_w64(acc[4 * q4 + e] <= tfj);
                    }
                    if (!(hit[0] | hit[1] | hit[2] | hit[3])) continue;
                    const uint4 pw = *reinterpret_cast<const uint4 *>(&xw[pb][rb0 + rb]);
                    const uint32_t wv[4] = {pw.x, pw.y, pw.z, pw.w};
#pragma unroll
                    for (int e = 0; e < 4; e++) {
                        if (!((hit[e] >> lane) & 1ull) || (wv[e] & my_mask) != my_val) continue;
                        const uint64_t key = ((uint64_t)f2ord(canon0(acc[4 * q4 + e])) << 32) | (uint32_t)(c0 + rb + e);
                        if (key < lst[MH - 1]) offer(key);
                    }
                }
                return;
            }
            // the elements at or below the bound whose packed words pass, as a mask
            uint32_t cand = 0;
            float least = inf;   // one key a lane: the least passing score
#pragma unroll
            for (int q4 = 0; q4 < 4; q4++) {
                const int rb = rb0 + 8 * q4 + 4 * g;
                const float4 pn = *reinterpret_cast<const float4 *>(&xn[pb][rb]);
                const uint4 pw = *reinterpret_cast<const uint4 *>(&xw[pb][rb]);
                const float pv[4] = {pn.x, pn.y, pn.z, pn.w};
                const uint32_t wv[4] = {pw.x, pw.y, pw.z, pw.w};
#pragma unroll
                for (int e = 0; e < 4; e++) {
                    const float sc = fmaf(cm, acc[4 * q4 + e], pv[e]);
                    acc[4 * q4 + e] = sc;
                    const bool in = sc <= tfj && (wv[e] & my_mask) == my_val;
                    cand |= in ? 1u << (4 * q4 + e) : 0u;
                    if (!LAB && MH == 1) least = fminf(least, in ? sc : inf);
                }
            }
            if constexpr (LAB && !DISJ) {
                // the signatures of all sixteen at once: until a lane's list is
                // full every score passes, and one at a time the lane with
                // most candidates keeps the wave waiting
                uint32_t sok = 0;
#pragma unroll
                for (int q4 = 0; q4 < 4; q4++) {
                    const uint64_t *sg = &xsig[pb][rb0 + 8 * q4 + 4 * g];
#pragma unroll
                    for (int e = 0; e < 4; e++) sok |= (my_lsig & ~sg[e]) == 0 ? 1u << (4 * q4 + e) : 0u;
                }
                cand &= sok;
            } else if constexpr (LAB) {   // the signatures and the terms of disjunctions
                for (uint32_t c = cand; c; c &= c - 1u) {
                    const int i = __builtin_ctz(c), row = rb0 + 8 * (i >> 2) + 4 * g + (i & 3);
                    if (!staged_passes(DISJ ? xw[pb][row] : 0u, !DISJ || has_lab ? xsig[pb][row] : ~0ull))
                        cand &= ~(1u << i);
                }
            } else if constexpr (MH == 1) {   // only the first of the least elements can enter
                uint32_t first = 0;
#pragma unroll
                for (int e = 0; e < 16; e++) first |= acc[e] == least ? 1u << e : 0u;
                cand &= first;
                cand &= 0u - cand;
            }
            while (cand) {
                const int r = __builtin_ctz(cand);
                cand &= cand - 1u;
                float sc = acc[0];
#pragma unroll
                for (int e = 1; e < 16; e++) sc = r == e ? acc[e] : sc;
                if (!LAB && MH == 1) sc = least;
                const uint32_t pos = (uint32_t)(c0 + 8 * (r >> 2) + 4 * g + (r & 3));
                const uint64_t key = ((uint64_t)f2ord(canon0(sc)) << 32) | pos;
                if (!(key < lst[MH - 1])) continue;
                if constexpr (LAB) {
                    if (has_lab && narrow && !my_or) {   // the labels against the staged slots
                        const uint4 sl = *reinterpret_cast<const uint4 *>(scur + (rb0 + pos - c0) * kMaxLabels);
                        uint4 ql = qlab[kXQ * w + c32];
                        bool ok = true;
                        for (int i = 0; i < my_nlab; i++) {   // (two labels a word)
                            const uint32_t v = (ql.x & 0xFFFFu) * 0x10001u;
                            const uint32_t x0 = sl.x ^ v, x1 = sl.y ^ v, x2 = sl.z ^ v, x3 = sl.w ^ v;
                            const uint32_t lo = min(min(x0 & 0xFFFFu, x1 & 0xFFFFu), min(x2 & 0xFFFFu, x3 & 0xFFFFu));
                            const uint32_t hi = min(min(x0 >> 16, x1 >> 16), min(x2 >> 16, x3 >> 16));
                            ok &= min(lo, hi) == 0u;
                            ql.x = ql.x >> 16 | ql.y << 16;
                            ql.y = ql.y >> 16 | ql.z << 16;
                            ql.z = ql.z >> 16 | ql.w << 16;
                            ql.w >>= 16;
                        }
                        if (!ok) continue;
                    } else if (has_lab && !rest_passes(my_qq, pos)) {   // (dense terms only: tested)
                        continue;
                    }
                }
                offer(key);
            }
        } else {
            if (j != lj) {   // level changed: the query's bound if it selects the level, NaN if not
                lj = j;
                tfj = ((my_sel >> j) & 1u) ? my_tf : qnan;
            }
            // The elements whose score passes the bound and whose packed word
            // passes the query's test, as a mask.  With labels nearly every
            // block has some; without, whether any score passes is found first.
            uint32_t cand = 0;
            float best = inf;   // (a NaN, of a masked row, is never the least)
#pragma unroll
            for (int q4 = 0; q4 < 4; q4++) {   // points 8 q4 + 4 g + e of the chunk, e < 4
                const float4 pn = *reinterpret_cast<const float4 *>(&xn[pb][rb0 + 8 * q4 + 4 * g]);
                const uint4 pw = LAB ? *reinterpret_cast<const uint4 *>(&xw[pb][rb0 + 8 * q4 + 4 * g]) : uint4{};
                const float pv[4] = {pn.x, pn.y, pn.z, pn.w};
                const uint32_t wv[4] = {pw.x, pw.y, pw.z, pw.w};
#pragma unroll
                for (int e = 0; e < 4; e++) {   // the element test's scores (deferred with their pairs)
                    const float sc = fmaf(cm, acc[4 * q4 + e], pv[e]);
                    acc[4 * q4 + e] = sc;
                    const uint32_t diff = (wv[e] & my_mask) ^ my_val;
                    if (LAB) cand |= sc <= tfj && diff == 0u ? 1u << (4 * q4 + e) : 0u;
                    else best = fminf(best, sc);
                }
            }
            if (!LAB) {
                if (!__builtin_amdgcn_ballot_w64(best <= tfj)) return;
#pragma unroll
                for (int q4 = 0; q4 < 4; q4++) {
                    const uint4 pw = *reinterpret_cast<const uint4 *>(&xw[pb][rb0 + 8 * q4 + 4 * g]);
                    const uint32_t wv[4] = {pw.x, pw.y, pw.z, pw.w};
#pragma unroll
                    for (int e = 0; e < 4; e++)
                        cand |= acc[4 * q4 + e] <= tfj && (wv[e] & my_mask) == my_val ? 1u << (4 * q4 + e) : 0u;
                }
            }
            // then lane by lane the lowest one at a time (few blocks have more
            // than one pass): the label signatures, and the ring
            if constexpr (LAB) {
                for (uint32_t c = cand; c; c &= c - 1u) {
                    const int i = __builtin_ctz(c), row = rb0 + 8 * (i >> 2) + 4 * g + (i & 3);
                    if (!staged_passes(DISJ ? xw[pb][row] : 0u, !DISJ || has_lab ? xsig[pb][row] : ~0ull))
                        cand &= ~(1u << i);
                }
            }
            for (uint64_t hm; (hm = __builtin_amdgcn_ballot_w64(cand != 0u)) != 0;) {
                const int n = __popcll(hm);   // at most 64
                if (vhead - vtail + n > kXRing) drain(vhead - vtail);
                if (cand) {
                    const int i = __builtin_ctz(cand);
                    cand &= cand - 1u;
                    float sc = acc[0];
#pragma unroll
                    for (int e = 1; e < 16; e++) sc = i == e ? acc[e] : sc;
                    const int sl = (vhead + __popcll(hm & lanemask_lt())) & (kXRing - 1);
                    ring_pos[sl] = (uint32_t)(c0 + 8 * (i >> 2) + 4 * g + (i & 3));
                    ring_row[sl] = (uint8_t)c32;
                    ring_key[sl] = f2ord(canon0(sc));
                }
                vhead += n;
            }
        }
    };
    auto step = [&](const uint8_t *cur, uint8_t *nxt, const uint16_t *scur, uint16_t *snxt, const int pb,
                    float (*nraw)[GR], const uint32_t *nsig, const float *nsc, float (*fraw)[GR], uint32_t *fsig,
                    float *fsc) -> bool {
        __builtin_amdgcn_s_waitcnt(0x0F70);   // vmcnt(0): the group's rows
        lds_barrier();
        if (x + 3 * kXG > cb + 64) plan(x);
        fetch_rows(x + kXG, nxt, snxt);
        fetch_points(x + 2 * kXG, fraw, fsig, fsc);
        {
            const int ci = pb ? w - kXG : w;   // the waves take turns
            if (ci >= 0 && ci < kXG) {
                const uint32_t jc = chunkj(x + kXG + ci);
                if (jc) point_terms(nraw, nsig, nsc, ci, (int)(jc >> 8), pb ^ 1);
            }
        }
        if (kXQ * w < nqt) {   // a wave without queries (small batches) only stages
#pragma unroll 1
            for (int i = 0; i < kXG; i++) {
                const uint32_t jc = chunkj(x + i);
                if (!jc) break;
                score(cur, scur, pb, i, chunk0(x + i), (int)(jc & 255u), (int)(jc >> 8));
            }
        }
        x += kXG;
        return chunkj(x) != 0;
    };
    while (step(xb0, xb1, xl0, xl1, 0, rw1, rg1, rs1, rw0, rg0, rs0) &&
           step(xb1, xb0, xl1, xl0, 1, rw0, rg0, rs0, rw1, rg1, rs1)) {
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
