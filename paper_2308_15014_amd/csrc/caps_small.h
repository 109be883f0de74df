// Small batches: declarations shared by caps_small.hip and the search.
#pragma once

#include "caps_internal.h"

namespace caps {

constexpr int kSmallQ = 256;                 // queries at most
// partitions, rounded up to a whole number on each of the 8 XCDs
__host__ __device__ constexpr int small_padded(int b) { return (b + 7) / 8 * 8; }
constexpr uint32_t kSmallSeed = 1u << 30;    // word of a (query, partition): level mask, slot << 16, seed probe

struct FrontArgs {
    const float *q;
    int32_t d;
    const int32_t *con_off, *con_attr, *con_val;
    int32_t n_con;
    Schema sch;
    int32_t disj;
    const float *cent, *cnorm;
    const float *scores;          // centroid scores nq x b (null: computed from cent in FP32)
    int32_t b, metric, m, s;      // s: seed probes in the first slots (s >= m: every probe)
    const int32_t *tags, *offs;
    int32_t h, rule;
    QDesc *qd, *qterms;
    int32_t *probes;
    uint32_t *sel;
    int32_t *cand, *ncand, *nsurv;
    uint64_t *tau;
    int32_t *dcnt, *oflow, *bad;
    void *qlow;                   // rounded queries (null: none), in format prec
    float *qscale, *qaux;
    int32_t dpad, prec;
    uint32_t *pmask;              // nq x b words (null: none)
    int32_t *cursor;              // two, cleared: the entry cursors of k_small_tiles
};

// One scan round's tiles: entries of the seed probes (which 1), the others (2)
// or all (0), tiles of qb entries, each written `split` times.
struct SmallRound {
    int32_t *entries;             // up to nq x m (null: no such round)
    uint32_t *esel;
    int4 *tiles;                  // small_padded(b) x ceil(nq / qb) x split
    int32_t which, qb, split;
};

struct DirectArgs {
    const int32_t *probes;
    const uint32_t *sel;
    const QDesc *qd, *qterms;
    const int32_t *offs, *perm;
    const float *vecs, *q;
    const uint32_t *words;
    const uint64_t *sigs;
    const uint16_t *slots;
    int32_t lslots, d, m, h, k, metric;
    uint64_t *partials;           // nq x m lists of k keys
    int32_t *nsurv;
};

bool small_fits(int32_t b, int32_t d, int32_t nq);
bool direct_fits(const IndexData *ix, int32_t nq, int32_t m);
caps_status small_front(const FrontArgs &A, int32_t nq, int device, hipStream_t st);
caps_status small_tiles(const uint32_t *pmask, int32_t nq, int32_t b, int32_t m, const SmallRound &r0,
                        const SmallRound &r1, int32_t *cursor, int device, hipStream_t st);
caps_status small_direct(const DirectArgs &A, int32_t nq, int32_t *ids, float *dist, hipStream_t st);

}  // namespace caps
