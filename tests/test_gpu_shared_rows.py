"""Large batches over few partitions, whose tiles' rows are shared by several
workgroups: exact results against the oracle with seed lists of two and eight
keys per workgroup, partitions with fewer chunks than workgroups, partitions
that hold nearly every row, lists that overflow, counters."""
import numpy as np
import pytest

import synth

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
    # seed, prec, n, d, b, h, metric, vocabs, label_vocab, disjunctive, k, m, one large partition
    (1700, "bf16", 12_000, 32, 9, 2, 0, (3, 4), 0, False, 10, 4, False),    # two keys, five shares
    (1701, "fp8", 12_000, 64, 9, 1, 0, (3,), 0, False, 40, 5, False),       # eight keys, five shares
    (1702, "fp16", 12_000, 128, 12, 0, 1, (), 9, False, 10, 3, False),      # labels
    (1703, "fp8", 12_000, 100, 12, 2, 1, (3,), 9, True, 12, 12, False),     # disjunctions
    (1704, "bf16", 12_000, 24, 40, 2, 0, (3,), 0, False, 2, 6, True),       # partitions of one row
    (1705, "fp8", 12_000, 128, 40, 1, 0, (2,), 5, False, 10, 36, True),     # m >= 32
    (1706, "none", 30_000, 128, 9, 2, 0, (3, 4), 0, False, 20, 9, False),   # the search's own copy
    (1707, "bf16", 4_000, 128, 40, 3, 0, (3, 3), 0, False, 1, 7, False),    # fewer chunks than shares
]


@pytest.mark.parametrize("case", CASES)
def test_shared_rows_equal_oracle(caps, orc, case):
    seed, prec, n, d, b, h, metric, voc, lv, disj, k, m, skew = case
    w = synth.make_tiny(seed, n=n, d=d, n_q=500, vocabs=voc, label_vocab=lv, metric=metric, b=b, h=h, cmin=0, cmax=2)
    init = np.arange(b, dtype=np.int32)
    if skew:
        w.x[1:b] *= 50.0   # centroids of their own, far from the other rows
    co, ca, cv = w.con_off, w.con_attr, w.con_val
    if disj:
        co, ca, cv = synth.draw_disjunctions(np.random.default_rng(seed), w.n_q, n, w.dense, w.label_off, w.labels, 1, 3, 0, 2)
    oi = orc.build_from_workload(w, iters=0, init=init)
    ix = caps.Index.build(w.x, w.dense, w.dense_vocab, w.label_off, w.labels, lv, metric=metric, n_partitions=b, kmeans_iters=0,
                          aft_height=h, init_ids=init, precision=prec)
    r = orc.search(oi, w.q, co, ca, cv, k, m, disjunctive=disj)
    for nq in (257, 500):
        for counters in (False, True):
            got = [t.cpu().numpy() for t in ix.search(w.q[:nq], co[:nq + 1], ca, cv, k, m, disjunctive=disj, counters=counters)]
            assert np.array_equal(got[0], r.ids[:nq]), (nq, counters)
            assert np.array_equal(got[1].view(np.uint32), r.dist[:nq].view(np.uint32)), (nq, counters)
            if counters:
                assert np.array_equal(got[2], r.n_cand[:nq]) and np.array_equal(got[3], r.n_surv[:nq])
    if prec != "none":   # the approximate search: as one large batch and in small ones, which share rows by their own rule
        a = [t.cpu().numpy() for t in ix.search(w.q, co, ca, cv, k, m, mode=1, disjunctive=disj)]
        for q0 in range(0, 500, 100):
            s = ix.search(w.q[q0:q0 + 100], co[q0:q0 + 101], ca, cv, k, m, mode=1, disjunctive=disj)
            assert np.array_equal(a[0][q0:q0 + 100], s[0].cpu().numpy()) and np.array_equal(a[1][q0:q0 + 100], s[1].cpu().numpy())
    ix.close()
