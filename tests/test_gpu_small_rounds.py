"""Small batches in two rounds of tiles (32 probes or more, too many rows for the
direct scan): seed tiles with shared rows that bound the main pass, the plain
scan's second round, up to four tiles of a partition, against the oracle."""
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
    # seed, prec, d, b, h, metric, vocabs, label_vocab, disjunctive, k, modes
    (830, "none", 128, 48, 2, 0, (3, 4), 0, False, 10, (0,)),        # plain scan, below the copy's rule and above
    (831, "bf16", 128, 48, 2, 0, (3, 4), 0, False, 10, (0, 2)),
    (832, "fp8", 128, 41, 3, 1, (4,), 12, False, 7, (0,)),           # labels
    (833, "fp16", 100, 48, 1, 0, (3,), 10, True, 40, (0, 2)),        # OR terms, lists of eight keys
    (834, "bf16", 200, 50, 4, 1, (3, 3), 0, True, 10, (0,)),         # rows of 256 elements
]


@pytest.mark.parametrize("case", CASES)
def test_two_round_small_batches_equal_oracle(caps, orc, case):
    seed, prec, d, b, h, metric, voc, lv, disj, k, modes = case
    n = 60_000
    w = synth.make_tiny(seed, n=n, d=d, n_q=256, vocabs=voc, label_vocab=lv, metric=metric, b=b, h=h, cmin=0, cmax=2)
    co, ca, cv = w.con_off, w.con_attr, w.con_val
    if disj:
        co, ca, cv = synth.draw_disjunctions(np.random.default_rng(seed), w.n_q, n, w.dense, w.label_off, w.labels, 1, 3, 0, 2)
    oi = orc.build_from_workload(w, iters=1)
    ix = caps.Index.from_workload(w, kmeans_iters=1, precision=prec)
    for m in (32, b):
        r = orc.search(oi, w.q, co, ca, cv, k, m, disjunctive=disj)
        for q in (17, 65, 200, 256):
            assert q * m * (n / b) * d > 64e6   # (above the direct scan's rule)
            for mode in modes:
                for counters in (False, True):
                    got = [t.cpu().numpy() for t in ix.search(w.q[:q], co[:q + 1], ca[:co[q]], cv[:co[q]], k, m, mode=mode,
                                                              disjunctive=disj, counters=counters)]
                    assert np.array_equal(got[0], r.ids[:q]), (m, q, mode, counters)
                    assert np.array_equal(got[1].view(np.uint32), r.dist[:q].view(np.uint32)), (m, q, mode, counters)
                    if counters:
                        assert np.array_equal(got[2], r.n_cand[:q]) and np.array_equal(got[3], r.n_surv[:q])
    ix.close()
