"""The 32 x 32 matrix-core scan in every storage format, row length, filter kind
and seed-list length: exact results (ids and distance bits) against the oracle,
with tiles past 128 entries, ragged chunk tails and rings that fill inside a tile."""
import numpy as np
import pytest

import synth
from oracle import ref64

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def caps():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2308_15014_amd as caps
    caps.lib()
    return caps


CASES = [
    # seed, prec, d, metric, vocabs, label_vocab, max_labels, disjunctive, k, m
    (600, "fp8", 24, 0, (), 12, 8, False, 10, 12),      # one step per row
    (601, "fp8", 128, 1, (4, 5), 30, 8, True, 10, 12),  # OR terms over dense values and labels
    (602, "fp16", 33, 0, (3,), 200, 24, False, 5, 7),   # wide slot rows
    (603, "bf16", 100, 1, (), 6, 4, False, 33, 9),      # long seed lists (four keys per lane)
    (604, "fp16", 128, 0, (4, 3), 0, 8, True, 10, 12),  # disjunctions without labels
    (605, "fp8", 65, 0, (3, 3), 0, 8, False, 20, 12),   # FP8 without labels
    (606, "bf16", 128, 0, (2,), 3, 2, False, 64, 3),    # too few seed probes for the seed lists
    (607, "bf16", 31, 0, (2, 2), 5, 3, False, 1, 12),   # k = 1
]


@pytest.mark.parametrize("case", CASES)
def test_x32_equals_oracle(caps, orc, case):
    seed, prec, d, metric, voc, lv, ml, disj, k, m = case
    w = synth.make_tiny(seed, n=7001, d=d, n_q=301, vocabs=voc, label_vocab=lv, metric=metric, b=12, h=2, cmin=0, cmax=2,
                        max_labels=ml)
    co, ca, cv = w.con_off, w.con_attr, w.con_val
    if disj:
        co, ca, cv = synth.draw_disjunctions(np.random.default_rng(seed), w.n_q, w.n, w.dense, w.label_off, w.labels, 1,
                                             3, 0, 2)
    oi = orc.build_from_workload(w, iters=2)
    ix = caps.Index.from_workload(w, kmeans_iters=2, precision=prec)
    r = orc.search(oi, w.q, co, ca, cv, k, m, disjunctive=disj)
    for counters in (False, True):
        got = ix.search(w.q, co, ca, cv, k, m, disjunctive=disj, counters=counters)
        assert np.array_equal(got[0].cpu().numpy(), r.ids)
        assert np.array_equal(got[1].cpu().numpy().view(np.uint32), r.dist.view(np.uint32))
        if counters:
            assert np.array_equal(got[2].cpu().numpy(), r.n_cand) and np.array_equal(got[3].cpu().numpy(), r.n_surv)
    ix.close()


APPROX = [
    # seed, prec, vocabs, label_vocab, d, rerank, n_q
    (620, "bf16", (3,), 0, 32, 12, 300),
    (621, "fp16", (), 5, 64, 40, 300),       # label tests
    (622, "fp8", (2,), 0, 128, 5, 300),      # two keys a list
    (623, "bf16", (2,), 4, 100, 64, 90),     # small batch
]


@pytest.mark.parametrize("case", APPROX)
def test_approximate_deferral(caps, orc, case):
    """Mode 1 on binary vectors, whose approximate scores are known (exact in the
    two-byte formats) and tie in thousands: the candidates are the `rerank` smallest (score, CSR position),
    from the deferred lists or, for queries whose pairs overflow those, from
    the rescue pass."""
    seed, prec, voc, lv, d, rr, nq = case
    w = synth.make_tiny(seed, n=24_000, d=d, n_q=nq, vocabs=voc, label_vocab=lv, b=40, h=2, cmin=0, cmax=2, integer=True)
    w.x = (w.x > 3).astype(np.float32)
    w.q = (w.q > 3).astype(np.float32)
    w.x[0] = w.q[0] = 1.0
    ix = caps.Index.from_workload(w, kmeans_iters=1, precision=prec)
    perm = ix.export()["perm"]
    k = 5
    ids, dist = (t.cpu().numpy() for t in ix.search(w.q, w.con_off, w.con_attr, w.con_val, k, 40, mode=1, rerank=rr))
    xc = w.x[perm]
    nx = (xc * xc).sum(1)
    for i in range(nq):
        ok = ref64.valid_mask(w.dense, w.label_off, w.labels, ref64.pairs_of(w.con_off, w.con_attr, w.con_val, i), w.n_dense,
                              w.dense_vocab, w.label_vocab)[perm]
        pos = np.flatnonzero(ok)
        dot = (xc[pos] @ w.q[i]).astype(np.float32)
        if prec == "fp8":   # codes of 448, both FP32 scales applied in turn (exact products otherwise)
            s = np.float32(1.0) / np.float32(448.0)
            dot = (dot * np.float32(448.0 * 448.0) * s) * s
        score = (nx[pos].astype(np.float64) - 2.0 * dot).astype(np.float32)   # (one fused rounding)
        cand = pos[np.lexsort((pos, score))[:rr]]
        dd = ((xc[cand] - w.q[i]) ** 2).sum(1)
        o = np.lexsort((perm[cand], dd))[:k]
        n = len(o)
        assert np.array_equal(ids[i, :n], perm[cand][o]) and np.all(ids[i, n:] == -1), i
        assert np.array_equal(dist[i, :n], dd[o].astype(np.float32)), i
    ix.close()


LONG = [
    # seed, prec, d, vocabs, label_vocab: partitions of about 3,000 rows, more than the 64 chunks laid out at once
    (640, "fp8", 32, (), 40),              # signatures folded into 32 bits of the packed word
    (641, "fp16", 96, (4096, 4096), 40),   # into 8 bits
    (642, "bf16", 128, (5000, 5000), 40),  # 6 bits left: not folded
    (643, "bf16", 64, (3,), 0),            # no labels
]


@pytest.mark.parametrize("case", LONG)
def test_long_partitions(caps, orc, case):
    seed, prec, d, voc, lv = case
    w = synth.make_tiny(seed, n=9001, d=d, n_q=290, vocabs=voc, label_vocab=lv, b=3, h=2, cmin=0, cmax=2)
    oi = orc.build_from_workload(w, iters=1)
    ix = caps.Index.from_workload(w, kmeans_iters=1, precision=prec)
    r = orc.search(oi, w.q, w.con_off, w.con_attr, w.con_val, 10, 3)
    got = ix.search(w.q, w.con_off, w.con_attr, w.con_val, 10, 3)
    assert np.array_equal(got[0].cpu().numpy(), r.ids)
    assert np.array_equal(got[1].cpu().numpy().view(np.uint32), r.dist.view(np.uint32))
    ix.close()
