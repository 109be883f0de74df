"""Queries and points near the ends of the FP32 range: approximate search of
queries whose norms overflow, centroid scores that overflow."""
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


@pytest.mark.parametrize("prec,d,label_vocab", [("bf16", 48, 0), ("fp8", 100, 0), ("bf16", 200, 6), ("fp8", 33, 6)])
def test_approximate_search_does_not_depend_on_query_scale(caps, prec, d, label_vocab):
    """Mode 1, inner product: a power of two in the query changes neither its
    codes' ratios nor any rounding, so ids are the same and scores scale, also
    where |q|^2 overflows."""
    w = synth.make_tiny(1200 + d, n=20_000, d=d, n_q=300, vocabs=(3,), label_vocab=label_vocab, metric=1, b=40, h=2, cmin=0, cmax=1)
    ix = caps.Index.from_workload(w, kmeans_iters=1, precision=prec)
    big = np.float32(2.0) ** 63
    assert np.all((w.q.astype(np.float64) ** 2).sum(1) * float(big) ** 2 > 3.5e38)
    for m in (7, 33, 40):
        for n in (90, 300):
            args = (w.con_off[:n + 1], w.con_attr[:w.con_off[n]], w.con_val[:w.con_off[n]])
            for kw in (dict(), dict(counters=True)):
                a = [t.cpu().numpy() for t in ix.search(w.q[:n], *args, 10, m, mode=1, **kw)]
                b = [t.cpu().numpy() for t in ix.search(w.q[:n] * big, *args, 10, m, mode=1, **kw)]
                assert np.array_equal(a[0], b[0]), (m, n, kw)
                assert np.array_equal((a[1] * big).view(np.uint32), b[1].view(np.uint32)), (m, n, kw)
            pa, pb = (ix.probes(q, *args, m, mode=1)[0].cpu().numpy() for q in (w.q[:n], w.q[:n] * big))
            assert np.array_equal(pa, pb)
    ix.close()


def test_overflowing_centroid_scores(caps, orc):
    """|c|^2 - 2 x.c with the product doubled before the subtraction: where it
    overflows alone the score is -inf, as the oracle computes it, and ties go to
    the smaller partition (assignment and routing, large and small batches)."""
    w = synth.make_tiny(1210, n=4000, d=8, n_q=300, vocabs=(3,), b=30, h=1, cmin=0, cmax=1)
    for t in (w.x, w.q):
        t[:, 0] = np.where(t[:, 0] < 0, -1.0, 1.0) * (1.35e19 + 1e17 * np.abs(t[:, 0]))   # (x.c)^2 < 3.4e38 < 2 x.c
    ids = np.arange(30, dtype=np.int32)
    oi = orc.build_from_workload(w, iters=0, init=ids)
    ix = caps.Index.build(w.x, w.dense, w.dense_vocab, metric=0, n_partitions=30, kmeans_iters=0, aft_height=1, init_ids=ids)
    assert len(np.unique(oi.assign)) < 30   # (scores of -inf tie)
    assert np.array_equal(ix.export()["assign"], oi.assign)
    for m in (1, 4):
        r = orc.search(oi, w.q, w.con_off, w.con_attr, w.con_val, 5, m)
        for n in (20, 300):
            pr = ix.probes(w.q[:n], w.con_off[:n + 1], w.con_attr, w.con_val, m)[0].cpu().numpy()
            assert np.array_equal(pr, r.probes[:n])
            got = ix.search(w.q[:n], w.con_off[:n + 1], w.con_attr, w.con_val, 5, m)
            assert np.array_equal(got[0].cpu().numpy(), r.ids[:n])
    ix.close()
