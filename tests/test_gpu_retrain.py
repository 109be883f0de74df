"""Training again on an index that has a router: the weights follow from the
parameters alone, whichever router was there before."""
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


def test_trainings_do_not_depend_on_earlier_ones(caps):
    w = synth.make_tiny(1600, n=3000, d=20, n_q=500, vocabs=(3, 4), b=24, h=1, cmin=0, cmax=2)
    labels = np.random.default_rng(1).integers(0, 24, (500, 3)).astype(np.int32)
    args = (w.q, w.con_off, w.con_attr, w.con_val)
    want = {}
    for hidden in (64, 96):
        for seed in (1, 2):
            ix = caps.Index.from_workload(w, kmeans_iters=1)
            loss = ix.router_train(*args, labels, hidden=hidden, epochs=2, batch=128, seed=seed)
            want[hidden, seed] = (ix.router_get(), loss, ix.router_logits(*args))
            ix.close()
    ix = caps.Index.from_workload(w, kmeans_iters=1)
    steps = [(64, 1), (64, 2), (64, 1), "set", (64, 2), (96, 1), (96, 2), (96, 1), (64, 1), "more", (64, 2), (64, 1)]
    for step in steps:
        if step == "set":
            g = want[64, 1][0]
            ix.router_set(g["w1"], g["b1"], g["w2"], g["b2"], hidden=64)
            step = (64, 1)
        elif step == "more":   # one more epoch on the router that is there
            ix.router_train(*args, labels, hidden=64, epochs=1, batch=128, seed=3, reset=0)
            continue
        else:
            loss = ix.router_train(*args, labels, hidden=step[0], epochs=2, batch=128, seed=step[1])
            assert np.array_equal(np.asarray(loss), np.asarray(want[step][1])), step
        got = ix.router_get()
        for k in ("w1", "b1", "w2", "b2"):
            assert np.array_equal(got[k], want[step][0][k]), (step, k)
        a, b = (np.asarray(t.cpu()) if hasattr(t, "cpu") else np.asarray(t) for t in (ix.router_logits(*args), want[step][2]))
        assert np.array_equal(a, b), step
        ix.search(*args, 5, 6, routing=1)
    ix.close()
