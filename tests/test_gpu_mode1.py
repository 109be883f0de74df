"""Approximate search (mode 1): results do not depend on whether survivors are
counted, on the batch a query is in or on the scan that its pairs go through."""
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


def _check(caps, w, prec, k, m, rerank):
    ix = caps.Index.from_workload(w, kmeans_iters=1, precision=prec)
    args = (w.q, w.con_off, w.con_attr, w.con_val, k, m)
    a = [t.cpu().numpy() for t in ix.search(*args, mode=1, rerank=rerank)]
    c = [t.cpu().numpy() for t in ix.search(*args, mode=1, rerank=rerank, counters=True)]
    n = 70
    e = w.con_off[n]
    s = [t.cpu().numpy() for t in ix.search(w.q[:n], w.con_off[:n + 1], w.con_attr[:e], w.con_val[:e], k, m, mode=1, rerank=rerank)]
    assert np.array_equal(a[0], c[0]) and np.array_equal(a[1], c[1])
    assert np.array_equal(a[0][:n], s[0]) and np.array_equal(a[1][:n], s[1])
    # valid, distinct, sorted, and every query with candidates answered
    for i in range(0, w.n_q, 17):
        got = a[0][i][a[0][i] >= 0]
        assert len(set(got)) == len(got) == min(k, int(c[3][i]))
        assert np.all(np.diff(a[1][i][:len(got)]) * (1 if w.metric == 0 else -1) >= 0)
    ix.close()
    return a


@pytest.mark.parametrize("prec", ["bf16", "fp16", "fp8"])
@pytest.mark.parametrize("metric,label_vocab,d", [(0, 0, 128), (1, 0, 96), (1, 8, 64), (0, 8, 30)])
def test_counters_do_not_change_results(caps, prec, metric, label_vocab, d):
    w = synth.make_tiny(1300 + d, n=24_000, d=d, n_q=400, vocabs=(3,), label_vocab=label_vocab, metric=metric, b=40, h=2, cmin=0, cmax=1)
    _check(caps, w, prec, 10, 36, 10)


@pytest.mark.parametrize("metric,label_vocab", [(1, 0), (1, 5), (0, 0)])
def test_fp8_scores_round_alike_in_every_scan(caps, metric, label_vocab):
    """Points and queries that share their large coordinates and differ in small
    ones: the sums lie within a few units in the last place of each other, and
    which points are rescored depends on how each was rounded."""
    rng = np.random.default_rng(5)
    w = synth.make_tiny(1350, n=24_000, d=128, n_q=400, vocabs=(3,), label_vocab=label_vocab, metric=metric, b=40, h=1, cmin=0, cmax=1)
    small = rng.permutation(128) < 32
    for t in (w.x, w.q):   # E4M3 values of every exponent, the largest 448: the scale is 1
        row = rng.integers(8, 16, 128) * np.exp2(rng.integers(-9, 6, 128)) * rng.choice([-1.0, 1.0], 128)
        row = np.clip(row, -448.0, 448.0)
        t[:] = rng.integers(8, 16, t.shape) / 64.0 * rng.choice([-1.0, 1.0], t.shape)
        t[:, ~small] = row[~small]
        t[:, np.flatnonzero(~small)[0]] = 448.0
    _check(caps, w, "fp8", 10, 40, 10)
