"""Survivor counts of label tests and disjunctions on an FP32 index, at the line
between the plain scan and the search's own BF16 copy (32 probes, k = 16),
against the oracle."""
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


@pytest.mark.parametrize("metric,label_vocab,disj", [(0, 9, False), (1, 0, True), (0, 9, True)])
def test_counts_and_results_equal_oracle(caps, orc, metric, label_vocab, disj):
    n, d, b, nq = 30_000, 64, 40, 720
    w = synth.make_tiny(1800 + label_vocab, n=n, d=d, n_q=nq, vocabs=(3, 4), label_vocab=label_vocab, metric=metric, b=b, h=2, cmin=0, cmax=2)
    co, ca, cv = w.con_off, w.con_attr, w.con_val
    if disj:
        co, ca, cv = synth.draw_disjunctions(np.random.default_rng(3), nq, n, w.dense, w.label_off, w.labels, 1, 3, 0, 2)
    oi = orc.build_from_workload(w, iters=1)
    ix = caps.Index.from_workload(w, kmeans_iters=1)
    for m, k in ((31, 16), (32, 16), (31, 17), (32, 17)):
        assert nq * m / b >= 64 and nq * m / b * n * d >= 1e9   # (large enough for a copy)
        r = orc.search(oi, w.q, co, ca, cv, k, m, disjunctive=disj)
        got = [t.cpu().numpy() for t in ix.search(w.q, co, ca, cv, k, m, disjunctive=disj, counters=True)]
        assert np.array_equal(got[0], r.ids), (m, k)
        assert np.array_equal(got[1].view(np.uint32), r.dist.view(np.uint32)), (m, k)
        assert np.array_equal(got[2], r.n_cand) and np.array_equal(got[3], r.n_surv), (m, k)
    ix.close()
