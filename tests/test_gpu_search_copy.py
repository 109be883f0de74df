"""Large exact searches on an index without a low-precision copy prune with a
BF16 copy made in the call's workspace: the results equal the oracle's and the
plain scan's (mode 2) bit for bit, also where norms overflow or underflow, and
smaller batches and budgets take the plain scan."""
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
    # seed, n, d, n_q, metric, vocabs, label_vocab, disjunctive, k, m of 16, extreme rows
    (700, 20_003, 128, 500, 0, (5, 6), 0, False, 10, 16, False),
    (701, 20_001, 33, 1700, 1, (4,), 30, False, 20, 16, False),     # scalar loads, labels
    (702, 15_000, 160, 450, 0, (3, 3), 0, True, 50, 16, False),     # 256-element rows
    (703, 20_000, 64, 1000, 0, (40, 30), 0, False, 10, 16, True),
    (704, 20_000, 64, 1000, 1, (40, 30), 12, False, 10, 14, True),
]


@pytest.mark.parametrize("case", CASES)
def test_copy_search_equals_plain_scan(caps, orc, case):
    seed, n, d, n_q, metric, voc, lv, disj, k, m, extreme = case
    w = synth.make_tiny(seed, n=n, d=d, n_q=n_q, vocabs=voc, label_vocab=lv, metric=metric, b=16, h=2, cmin=0, cmax=3)
    if extreme:   # |x|^2 that overflows, lies near overflow, underflows
        w.x[10:400:13] *= 1e20
        w.x[11:400:13] *= 3e18
        w.x[12:400:13] *= 1e-25
        w.q[3:60:7] *= 2e18 if metric == 0 else 1e10
        w.q[4:60:7] *= 1e-30
    co, ca, cv = w.con_off, w.con_attr, w.con_val
    if disj:
        co, ca, cv = synth.draw_disjunctions(np.random.default_rng(seed), n_q, n, w.dense, w.label_off, w.labels, 1, 3, 0, 2)
    ix = caps.Index.from_workload(w, kmeans_iters=2)
    dpad = 32 * (1 << max(0, (d - 1) // 32).bit_length())
    copied = ix.workspace_bytes(n_q, k, m)
    assert copied > ix.workspace_bytes(n_q, k, m, mode=2) + 2 * dpad * n
    assert ix.workspace_bytes(20, k, m) < 2 * dpad * n   # a small batch makes no copy
    args = (w.q, co, ca, cv, k, m)
    plain = [t.cpu().numpy() for t in ix.search(*args, mode=2, disjunctive=disj, counters=True)]
    for kw in (dict(), dict(counters=True), dict(workspace_bytes=copied // 2), dict(workspace_bytes=3 * copy_bytes(n, dpad))):
        got = [t.cpu().numpy() for t in ix.search(*args, disjunctive=disj, **kw)]
        for a, b in zip(got, plain):
            assert np.array_equal(a.view(np.uint32), b.view(np.uint32)), kw
    if not extreme:
        oi = orc.build_from_workload(w, iters=2)
        r = orc.search(oi, w.q, co, ca, cv, k, m, disjunctive=disj)
        assert np.array_equal(plain[0], r.ids) and np.array_equal(plain[1].view(np.uint32), r.dist.view(np.uint32))
    ix.close()


def copy_bytes(n, dpad):
    return n * (2 * dpad + 12)


def test_plain_scan_limits_hold(caps):
    """d = 200 with k = 50 exceeds the plain scan's LDS: refused for large
    batches, which would make a copy, as for small ones."""
    w = synth.make_tiny(710, n=15_000, d=200, n_q=400, vocabs=(3, 3), b=16, h=2)
    ix = caps.Index.from_workload(w, kmeans_iters=1)
    for n in (10, 400):
        with pytest.raises(caps.CapsError) as e:
            ix.search(w.q[:n], w.con_off[:n + 1], w.con_attr, w.con_val, 50, 16)
        assert e.value.status == -4
    ix.close()
