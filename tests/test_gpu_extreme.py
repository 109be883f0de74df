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
