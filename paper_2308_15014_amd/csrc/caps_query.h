// Device code shared by the search paths (internal): a query's filter
// descriptor, its sub-partition choice and the rounding of query rows.
#pragma once

#include <math.h>

#include "caps_device.h"
#include "caps_internal.h"

namespace caps {

// ------------------------------------------------------------------ filter
__device__ inline void qd_clear(QDesc &r) {
    r.dmask = 0;
    r.dval = 0;
    r.flags = 0;
    r.nlab = 0;
    r.lsig = 0;
    for (int i = 0; i < kMaxLabels; i++) r.lab[i] = 0xFFFF;
    r.nterm = 1;
    r.pad = 0;
}

// Adds constraint pair (a, v) to the AND-term r: a dense value becomes a
// packed field under dmask, a label joins the label list and signature; a
// pair outside the vocabularies, a second value of one dense attribute or a
// ninth label makes the term unsatisfiable.
__device__ inline void qd_add(QDesc &r, const Schema &sch, int32_t a, int32_t v) {
    if (a < 0 || a > sch.n_dense) {
        r.flags |= kQUnsat;
        return;
    }
    if (a < sch.n_dense) {
        if (v < 0 || v >= sch.dense_vocab[a]) {
            r.flags |= kQUnsat;
            return;
        }
        const uint32_t fm = (uint32_t)(((1ull << sch.field_bits[a]) - 1ull) << sch.field_shift[a]);
        const uint32_t fv = (uint32_t)v << sch.field_shift[a];
        if ((r.dmask & fm) && ((r.dval & fm) != fv)) r.flags |= kQUnsat;
        r.dmask |= fm;
        r.dval = (r.dval & ~fm) | fv;
        return;
    }
    if (sch.label_vocab == 0 || v < 0 || v >= sch.label_vocab) {
        r.flags |= kQUnsat;
        return;
    }
    for (int i = 0; i < r.nlab; i++)
        if (r.lab[i] == (uint16_t)v) return;   // duplicate: AND is idempotent
    if (r.nlab == kMaxLabels) {
        r.flags |= kQUnsat;
        return;
    }
    r.lab[r.nlab++] = (uint16_t)v;
    r.lsig |= 1ull << label_sig_bit((uint32_t)v);
}

// Summary of a disjunction of nsat > 1 satisfiable terms: the dense fields
// every term fixes to the same value.
__device__ inline void qd_summary(QDesc &r, const Schema &sch, const QDesc *tq, int nsat) {
    uint32_t all = ~0u, diff = 0;
    for (int t = 0; t < nsat; t++) {
        all &= tq[t].dmask;
        diff |= tq[t].dval ^ tq[0].dval;
    }
    uint32_t keep = 0;
    for (int a = 0; a < sch.n_dense; a++) {
        const uint32_t fm = (uint32_t)(((1ull << sch.field_bits[a]) - 1ull) << sch.field_shift[a]);
        if ((all & fm) == fm && !(diff & fm)) keep |= fm;
    }
    r.dmask = keep;
    r.dval = tq[0].dval & keep;
    r.flags = kQOr;
    r.nterm = nsat;
}

// The pairs [lo, hi) as a disjunction, terms separated by CAPS_OR: the
// satisfiable terms go to tq, r (clear before) becomes their summary (one
// satisfiable term: that term; none, or more than kMaxTerms terms:
// unsatisfiable).  cur: scratch.
__device__ inline void qd_disjunction(QDesc &r, QDesc &cur, QDesc *tq, const Schema &sch, const int32_t *attr,
                                      const int32_t *val, int32_t lo, int32_t hi) {
    qd_clear(cur);
    int nt = 0, nsat = 0;
    for (int32_t e = lo; e <= hi; e++) {
        if (e < hi && attr[e] != CAPS_OR) {
            qd_add(cur, sch, attr[e], val[e]);
            continue;
        }
        if (++nt > kMaxTerms) break;
        if (!(cur.flags & kQUnsat)) tq[nsat++] = cur;
        qd_clear(cur);
    }
    if (nt > kMaxTerms || nsat == 0) r.flags |= kQUnsat;
    else if (nsat == 1) r = tq[0];
    else qd_summary(r, sch, tq, nsat);
}

// ------------------------------------------------------------------ sub-partition choice
__device__ inline void tag_decode(const Schema &s, int32_t tok, int &attr, int32_t &val) {
    if (tok < s.dense_off[s.n_dense]) {
        int a = 0;
        while (a + 1 < s.n_dense && tok >= s.dense_off[a + 1]) a++;
        attr = a;
        val = tok - s.dense_off[a];
    } else {
        attr = s.n_dense;
        val = tok - s.dense_off[s.n_dense];
    }
}

// Exact rule: J* = first tagged level whose tag the query holds (h if none);
// scan level j < h iff j <= J*, tagged, and its tag does not contradict a
// dense constraint; scan the remainder iff J* = h.  rule 1: only level J*.
__device__ inline uint32_t choose_levels(const Schema &s, const QDesc &qd, const int32_t *tags, int h,
                                         int rule) {
    if (qd.flags & (kQUnsat | kQNonFinite)) return 0u;
    int js = h;
    uint32_t ok = 0;
    for (int j = 0; j < h; j++) {
        const int32_t t = tags[j];
        if (t < 0) continue;
        int a;
        int32_t v;
        tag_decode(s, t, a, v);
        bool held, conflict = false;
        if (a < s.n_dense) {
            const uint32_t fm = (uint32_t)(((1ull << s.field_bits[a]) - 1ull) << s.field_shift[a]);
            const bool constrained = (qd.dmask & fm) != 0;
            const bool same = ((qd.dval & fm) >> s.field_shift[a]) == (uint32_t)v;
            held = constrained && same;
            conflict = constrained && !same;
        } else {
            held = false;
            for (int i = 0; i < qd.nlab; i++) held |= qd.lab[i] == (uint16_t)v;
        }
        if (!conflict) ok |= 1u << j;
        if (held) {
            js = j;
            break;
        }
    }
    if (rule == 1) return 1u << js;
    uint32_t mask = ok & ((js >= 31) ? 0xFFFFFFFFu : ((2u << js) - 1u));
    if (js == h) mask |= 1u << h;
    return mask;
}

// A query's levels: the union over its terms for a disjunction (Section 5.3:
// several sub-partitions per partition join the candidate set).
__device__ inline uint32_t choose_query_levels(const Schema &s, const QDesc &qd, const QDesc *terms,
                                               const int32_t *tags, int h, int rule) {
    if (qd.flags & (kQUnsat | kQNonFinite)) return 0u;
    if (!(qd.flags & kQOr)) return choose_levels(s, qd, tags, h, rule);
    uint32_t mask = 0;
    for (int t = 0; t < qd.nterm; t++) mask |= choose_levels(s, terms[t], tags, h, rule);
    return mask;
}

// ------------------------------------------------------------------ rounding
__device__ inline uint16_t f16_rne_sat(float f) {
    f = fminf(fmaxf(f, -65504.0f), 65504.0f);
    return __builtin_bit_cast(uint16_t, (_Float16)f);
}

// OCP E4M3 (bias 7, max 448, 0x7F/0xFF are NaN): round to nearest even,
// saturating to +-448.
__device__ inline uint8_t e4m3_rne_sat(float v) {
    const uint8_t sign = v < 0.0f ? 0x80 : 0x00;
    const float a = fabsf(v);
    if (!(a < 448.0f)) return sign | 0x7E;
    if (a < 0.015625f) {   // below the smallest normal 2^-6: quantum 2^-9
        const int qi = (int)rintf(a * 512.0f);
        return qi == 0 ? (uint8_t)0 : (uint8_t)(sign | qi);   // single zero; 8 is the smallest normal
    }
    int e2;
    (void)frexpf(a, &e2);
    int e = e2 - 1;                       // a in [2^e, 2^(e+1))
    int q = (int)rintf(ldexpf(a, 3 - e)); // in [8, 16]
    if (q == 16) {
        e += 1;
        q = 8;
    }
    return sign | (uint8_t)(((e + 7) << 3) | (q - 8));
}

// Value of an E4M3 code (finite codes only).
__device__ inline double e4m3_value(uint8_t c) {
    const int e = (c >> 3) & 15, m = c & 7;
    const double v = e == 0 ? ldexp((double)m, -9) : ldexp((double)(8 + m), e - 10);
    return (c & 0x80) ? -v : v;
}

// FP64 -> FP32 rounded towards +inf / -inf (inputs >= 0).
__device__ inline float f32_up(double v) {
    const float f = (float)v;
    return (double)f < v ? nextafterf(f, __builtin_huge_valf()) : f;
}
__device__ inline float f32_down(double v) {
    const float f = (float)v;
    return (double)f > v ? nextafterf(f, 0.0f) : f;
}

// relative slack covering the FP64 sums and square roots of the error norms
constexpr double kNormSlack = 1.0 + 0x1p-40;

// Above this |x|^2 (FP32 overflow is near) a query of an exact search, or a row
// of the BF16 copy that a search makes for itself, gets zero codes and infinite
// error norms: its pairs always pass the bound and are rescored.  (Not the rows
// of an index's own copy, nor the queries of the approximate search, whose
// scores have no bound to fall back on.)
constexpr float kNormMax = 1e37f;

// One wave, query row r (the i-th): rounded copy (the codes of k_quantize, element by
// element), FP8 scale and qaux = {|q| (up), |q|^2 (down), |q - q~| (up),
// |q~| (up)}; the FP64 sums are reduced across the wave (their order does
// not matter: kNormSlack covers any order).  exact: for the exact search's
// bound; the approximate search keeps the codes of every query.
__device__ inline void qquant_row(const float *__restrict__ r, int64_t i, int32_t d, int32_t dpad, int32_t prec, bool exact,
                                  void *__restrict__ out, float *__restrict__ scale, float *__restrict__ qaux) {
    const int lane = threadIdx.x & 63;
    float s = 1.0f;
    if (prec == CAPS_PREC_FP8) {
        float amax = 0.0f;
        for (int j = lane; j < d; j += 64) amax = fmaxf(amax, fabsf(r[j]));
#pragma unroll
        for (int o = 32; o >= 1; o >>= 1) amax = fmaxf(amax, __shfl_xor(amax, o, 64));
        s = amax > 0.0f ? amax / 448.0f : 1.0f;
    }
    double e2 = 0.0, a2 = 0.0, n2 = 0.0;
    for (int j = lane; j < dpad; j += 64) {
        const float x = j < d ? r[j] : 0.0f;
        double v;
        if (prec == CAPS_PREC_FP8) {
            const uint8_t c = j < d ? e4m3_rne_sat(x / s) : (uint8_t)0;
            reinterpret_cast<uint8_t *>(out)[i * dpad + j] = c;
            v = (double)s * e4m3_value(c);
        } else {
            const uint16_t c = j < d ? (prec == CAPS_PREC_BF16 ? bf16_rne(x) : f16_rne_sat(x)) : (uint16_t)0;
            reinterpret_cast<uint16_t *>(out)[i * dpad + j] = c;
            v = prec == CAPS_PREC_BF16 ? (double)__builtin_bit_cast(float, (uint32_t)c << 16)
                                       : (double)__builtin_bit_cast(_Float16, c);
        }
        if (j < d) {
            e2 += ((double)x - v) * ((double)x - v);
            a2 += v * v;
            n2 += (double)x * (double)x;
        }
    }
#pragma unroll
    for (int o = 32; o >= 1; o >>= 1) {
        e2 += __shfl_xor(e2, o, 64);
        a2 += __shfl_xor(a2, o, 64);
        n2 += __shfl_xor(n2, o, 64);
    }
    double nlo = n2 / kNormSlack;
    // near FP32 overflow: zero codes and an infinite error norm, as for a row of
    // that size (an infinite code times a zero would make a NaN score, which
    // never passes)
    if (exact && !(n2 < (double)kNormMax && a2 < (double)kNormMax)) {
        for (int j = lane; j < dpad; j += 64) {
            if (prec == CAPS_PREC_FP8)
                reinterpret_cast<uint8_t *>(out)[i * dpad + j] = 0;
            else
                reinterpret_cast<uint16_t *>(out)[i * dpad + j] = 0;
        }
        e2 = __builtin_huge_val();
        nlo = 0.0;   // (a finite lower bound on |q|^2)
    }
    if (lane == 0) {
        scale[i] = s;
        qaux[4 * i + 0] = f32_up(sqrt(n2) * kNormSlack);
        qaux[4 * i + 1] = f32_down(nlo);
        qaux[4 * i + 2] = f32_up(sqrt(e2) * kNormSlack);
        qaux[4 * i + 3] = f32_up(sqrt(a2) * kNormSlack);
    }
}

}  // namespace caps
