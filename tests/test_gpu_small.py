"""The small-batch path (front kernel, direct scan, tiles of small batches with
shared rows) against the oracle, at the edges of its rules: one query, the
largest small batch and one more, every storage format, ties of centroid scores,
unconstrained and non-finite queries, counters, probes and survivor masks."""
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
    # seed, prec, n, d, b, h, metric, vocabs, label_vocab, max_labels, disjunctive, k
    (800, "none", 9000, 37, 40, 2, 0, (3, 4), 0, 4, False, 10),      # scalar rows
    (801, "bf16", 60_000, 128, 24, 3, 0, (4, 6), 0, 4, False, 10),   # tiles with shared rows
    (802, "fp8", 60_000, 96, 24, 4, 1, (), 20, 8, False, 5),         # labels
    (803, "fp16", 50_000, 64, 24, 1, 0, (3,), 30, 24, True, 12),     # wide labels, OR terms
    (804, "bf16", 40_000, 200, 20, 0, 0, (3, 3), 0, 4, True, 64),    # long rows, longest list
    (805, "none", 3000, 20, 1100, 2, 0, (2,), 0, 4, False, 3),       # more partitions than threads
    (806, "none", 50_000, 100, 30, 2, 1, (3, 3), 6, 4, False, 50),   # plain scan, two rounds
]


@pytest.mark.parametrize("case", CASES)
def test_small_batches_equal_oracle(caps, orc, case):
    import torch
    seed, prec, n, d, b, h, metric, voc, lv, ml, disj, k = case
    nq = 257
    w = synth.make_tiny(seed, n=n, d=d, n_q=nq, vocabs=voc, label_vocab=lv, metric=metric, b=b, h=h, cmin=0, cmax=2,
                        max_labels=ml)
    w.x[: n // 2] = np.rint(w.x[: n // 2] * 2)   # (ties of distances)
    co, ca, cv = w.con_off, w.con_attr, w.con_val
    if disj:
        co, ca, cv = synth.draw_disjunctions(np.random.default_rng(seed), nq, n, w.dense, w.label_off, w.labels, 1, 3, 0, 2)
    oi = orc.build_from_workload(w, iters=2)
    ix = caps.Index.from_workload(w, kmeans_iters=2, precision=prec)
    for m in (1, b // 3, b):
        r = orc.search(oi, w.q, co, ca, cv, k, m, disjunctive=disj)
        for q in (1, 3, 64, 65, 200, 256, 257):
            args = (w.q[:q], co[:q + 1], ca[:co[q]], cv[:co[q]], k, m)
            for kw in (dict(), dict(counters=True, mode=2 if prec == "bf16" else 0)):
                if kw.get("mode") == 2 and k == 64:
                    continue   # (the plain scan's LDS limit)
                got = ix.search(*args, disjunctive=disj, **kw)
                torch.cuda.synchronize()
                assert np.array_equal(got[0].cpu().numpy(), r.ids[:q]), (m, q, kw)
                assert np.array_equal(got[1].cpu().numpy().view(np.uint32), r.dist[:q].view(np.uint32)), (m, q, kw)
                if len(got) > 2:
                    assert np.array_equal(got[2].cpu().numpy(), r.n_cand[:q]), (m, q, kw)
                    assert np.array_equal(got[3].cpu().numpy(), r.n_surv[:q]), (m, q, kw)
    ix.close()


def test_small_tied_centroids_and_bad_rows(caps, orc):
    """Partitions in identical groups: the m-th centroid score is tied, the
    smaller ids are probed; a NaN row answers empty and leaves the others."""
    w = synth.make_tiny(810, n=6000, d=16, n_q=40, vocabs=(3, 4), b=1500, h=2, cmin=0, cmax=2, integer=True)
    w.x[:1500] = np.repeat(w.x[:50], 30, axis=0)   # initial centroids (ids below) in 50 groups of 30
    init = np.arange(1500, dtype=np.int32)
    oi = orc.build_from_workload(w, iters=0, init=init)
    ix = caps.Index.build(w.x, w.dense, w.dense_vocab, metric=0, n_partitions=1500, kmeans_iters=0, aft_height=2, init_ids=init)
    for m in (7, 31, 1499):
        r = orc.search(oi, w.q, w.con_off, w.con_attr, w.con_val, 10, m)
        pr, _ = ix.probes(w.q, w.con_off, w.con_attr, w.con_val, m)
        got = ix.search(w.q, w.con_off, w.con_attr, w.con_val, 10, m, counters=True)
        assert np.array_equal(np.sort(pr.cpu().numpy(), 1), np.sort(r.probes, 1))
        assert np.array_equal(got[0].cpu().numpy(), r.ids) and np.array_equal(got[2].cpu().numpy(), r.n_cand)
        bad = w.q.copy()
        bad[5, 3] = np.nan
        bad[6, 0] = np.inf
        got = ix.search(bad, w.con_off, w.con_attr, w.con_val, 10, m)[0].cpu().numpy()
        keep = np.setdiff1d(np.arange(40), [5, 6])
        assert np.all(got[[5, 6]] == -1) and np.array_equal(got[keep], r.ids[keep])
        with pytest.raises(caps.CapsError):
            ix.search(bad, w.con_off, w.con_attr, w.con_val, 10, m, validate=True)
        ix.search(w.q, w.con_off, w.con_attr, w.con_val, 10, m, validate=True)
    ix.close()
