"""GPU learned router against the FP64 oracle (oracle/router.py) and its
behavioural contract: forward logits and batch gradients within 1e-4 of each
tensor's norm (same BF16 operand roundings on both sides); a router that
always falls back routes exactly like the centroids; training lowers the
loss; and on a workload whose filters point away from the query's nearest
clusters, learned routing finds more of the exact answers at a small nprobe."""
import numpy as np
import pytest

import synth
from oracle import router as R

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def caps():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2308_15014_amd as caps
    caps.lib()
    return caps


def _rel(a, b):
    a = np.asarray(a, np.float64)
    b = np.asarray(b, np.float64)
    return np.linalg.norm(a - b) / max(np.linalg.norm(b), 1e-30)


def _weights(rng, hid, dp, b):
    w = dict(w1=(rng.normal(size=(hid, dp)) * 0.15).astype(np.float32),
             b1=(rng.normal(size=hid) * 0.1).astype(np.float32),
             w2=(rng.normal(size=(b, hid)) * 0.15).astype(np.float32),
             b2=(rng.normal(size=b) * 0.1).astype(np.float32))
    return w


def _subset(w, idx):
    co = np.concatenate([[0], np.cumsum(np.diff(w.con_off)[idx])]).astype(np.int32)
    ca = np.concatenate([w.con_attr[w.con_off[i]:w.con_off[i + 1]] for i in idx]).astype(np.int32)
    cv = np.concatenate([w.con_val[w.con_off[i]:w.con_off[i + 1]] for i in idx]).astype(np.int32)
    return w.q[idx], co, ca, cv


@pytest.fixture(scope="module")
def tiny(caps):
    w = synth.make_tiny(300, n=1500, d=32, n_q=90, vocabs=(3, 5), label_vocab=20, b=16, h=2, cmin=0, cmax=3)
    ix = caps.Index.from_workload(w, kmeans_iters=3)
    return w, ix


def test_logits_match_oracle(caps, tiny):
    w, ix = tiny
    rng = np.random.default_rng(1)
    dp = R.pad_width(w.d)
    wt = _weights(rng, 64, dp, 16)
    ix.router_set(**wt, hidden=64, in_scale=0.5, in_shift=0.1)
    inf = ix.router_info()
    assert inf["present"] == 1 and inf["dpad"] == dp and inf["n_out"] == 16
    got = ix.router_logits(w.q, w.con_off, w.con_attr, w.con_val).cpu().numpy()
    x = R.input_rows(w.q, w.con_off, w.con_attr, w.con_val, w.dense_vocab, w.label_vocab, 0.5, 0.1)
    want, _ = R.forward(x, **wt)
    assert _rel(got, want) < 1e-4
    back = ix.router_get()
    for k in wt:
        assert np.array_equal(back[k], wt[k])


def test_gradients_match_oracle(caps, tiny):
    w, ix = tiny
    rng = np.random.default_rng(2)
    dp = R.pad_width(w.d)
    wt = _weights(rng, 48, dp, 16)
    ix.router_set(**wt, hidden=48, in_scale=0.7, in_shift=-0.2)
    labels = rng.integers(-1, 16, size=(w.n_q, 3)).astype(np.int32)
    loss, g = ix.router_grads(w.q, w.con_off, w.con_attr, w.con_val, labels)
    x = R.input_rows(w.q, w.con_off, w.con_attr, w.con_val, w.dense_vocab, w.label_vocab, 0.7, -0.2)
    want_loss, want = R.loss_and_grads(x, labels, **wt)
    assert abs(loss - want_loss) <= 1e-4 * abs(want_loss)
    for k in ("w1", "b1", "w2", "b2"):
        assert _rel(g[k], want[k]) < 1e-4, k


def test_always_fallback_is_centroid_routing(caps, tiny):
    w, ix = tiny
    rng = np.random.default_rng(3)
    ix.router_set(**_weights(rng, 32, R.pad_width(w.d), 16), hidden=32, fallback_prob=1.5)
    for m in (1, 5, 16):
        for mode in (0, 2):
            a = ix.search(w.q, w.con_off, w.con_attr, w.con_val, 7, m, mode=mode, routing=0, counters=True)
            b = ix.search(w.q, w.con_off, w.con_attr, w.con_val, 7, m, mode=mode, routing=1, counters=True)
            for x, y in zip(a, b):
                assert np.array_equal(x.cpu().numpy().view(np.uint32), y.cpu().numpy().view(np.uint32))
        pa, ma = ix.probes(w.q, w.con_off, w.con_attr, w.con_val, m, routing=0)
        pb, mb = ix.probes(w.q, w.con_off, w.con_attr, w.con_val, m, routing=1, k=7)
        assert np.array_equal(pa.cpu().numpy(), pb.cpu().numpy())


def test_partial_fallback_mixes_router_and_centroid_probes(caps, tiny):
    """Queries below the fallback level take the centroid probes, the others
    the router's top-m (unless their router probes hold fewer than k
    candidates): the centroid scores are computed for the falling-back
    queries only, on a compacted list."""
    w, ix = tiny
    rng = np.random.default_rng(4)
    ix.router_set(**_weights(rng, 32, R.pad_width(w.d), 16), hidden=32)
    z = ix.router_logits(w.q, w.con_off, w.con_attr, w.con_val).cpu().numpy().astype(np.float64)
    conf = 1.0 / np.exp(z - z.max(axis=1, keepdims=True)).sum(axis=1)
    cs = np.sort(conf)
    gaps = np.diff(cs)
    mid = len(cs) // 2
    j = mid - 5 + int(np.argmax(gaps[mid - 5:mid + 5]))   # the widest gap near the median
    assert gaps[j] > 1e-4 * cs[j]
    fb = 0.5 * (cs[j] + cs[j + 1])
    ix.router_set(**ix.router_get(), hidden=32, fallback_prob=float(fb))
    m = 5
    pc, _ = ix.probes(w.q, w.con_off, w.con_attr, w.con_val, m, routing=0)
    pr, _ = ix.probes(w.q, w.con_off, w.con_attr, w.con_val, m, routing=1, k=1)
    pc, pr = pc.cpu().numpy(), pr.cpu().numpy()
    n_router = 0
    for i in range(w.n_q):
        if conf[i] < fb:
            assert np.array_equal(pr[i], pc[i]), i
        else:
            key = sorted(range(z.shape[1]), key=lambda c: (-np.float32(z[i, c]), c))[:m]
            assert np.array_equal(pr[i], key) or np.array_equal(pr[i], pc[i]), i
            n_router += int(np.array_equal(pr[i], key))
    assert (conf < fb).sum() > 10 and n_router > 10


def test_labels_are_partitions_of_the_ids(caps, tiny):
    w, ix = tiny
    ids, _ = ix.search(w.q, w.con_off, w.con_attr, w.con_val, 10, 16)
    lab = ix.router_labels(ids).cpu().numpy()
    assign = ix.export()["assign"]
    for i, row in enumerate(ids.cpu().numpy()):
        want = []
        for v in row:
            if v >= 0 and assign[v] not in want:
                want.append(int(assign[v]))
        assert lab[i].tolist() == want + [-1] * (10 - len(want))


def test_learned_routing_gain(caps):
    w = synth.make_routed(n=40_000, n_q=6000, purity=1.0)
    ix = caps.Index.from_workload(w)
    b = w.n_partitions
    tr, te = np.arange(0, 5000), np.arange(5000, 6000)
    q, co, ca, cv = _subset(w, tr)
    truth, _ = ix.search(q, co, ca, cv, 10, b)
    labels = ix.router_labels(truth)
    loss = ix.router_train(q, co, ca, cv, labels, hidden=256, epochs=30, batch=256, lr=2e-3,
                           in_scale=1.0 / 3.0, seed=7)
    assert loss[-1] < 0.6 * loss[0]
    qt, cot, cat, cvt = _subset(w, te)
    tt, _ = ix.search(qt, cot, cat, cvt, 10, b)
    tt = tt.cpu().numpy()

    def recall(ids):
        ids = ids.cpu().numpy()
        return np.mean([len(set(a[a >= 0]) & set(t[t >= 0])) / max(1, (t >= 0).sum()) for a, t in zip(ids, tt)])

    m = 4
    r0 = recall(ix.search(qt, cot, cat, cvt, 10, m, routing=0)[0])
    r1 = recall(ix.search(qt, cot, cat, cvt, 10, m, routing=1)[0])
    assert r1 > r0 + 0.15, (r0, r1)


def test_adam_steps_match_oracle(caps, tiny):
    """k_adam against the Adam step of the oracle (bias-corrected, FP64)
    applied to the GPU's own batch gradient: three steps on one row each,
    the moments carried from step to step."""
    w, ix = tiny
    rng = np.random.default_rng(4)
    dp = R.pad_width(w.d)
    wt = _weights(rng, 32, dp, 16)
    lr, b1, b2, eps = 3e-3, 0.9, 0.999, 1e-8
    ix.router_set(**wt, hidden=32, in_scale=0.5, in_shift=0.0)
    labels = rng.integers(0, 16, size=(w.n_q, 2)).astype(np.int32)
    params = {k: v.astype(np.float64) for k, v in wt.items()}
    mom = {k: np.zeros_like(v) for k, v in params.items()}
    vel = {k: np.zeros_like(v) for k, v in params.items()}
    for step in (1, 2, 3):
        q, co, ca, cv = _subset(w, [step])
        lab = labels[step:step + 1]
        _, g = ix.router_grads(q, co, ca, cv, lab)
        ix.router_train(q, co, ca, cv, lab, hidden=32, epochs=1, batch=1, reset=0, lr=lr, beta1=b1, beta2=b2,
                        eps=eps, in_scale=0.5, in_shift=0.0)
        assert ix.router_info()["steps"] == step
        params = R.adam(params, g, mom, vel, step, lr, b1, b2, eps)
        got = ix.router_get()
        for k in params:
            want = params[k]
            # the GPU rounds each parameter to FP32 once per step and evaluates
            # the update (about lr in size) in FP32 from FP32 moments
            tol = 4 * step * np.spacing(np.abs(want).astype(np.float32)).astype(np.float64) + step * lr * 1e-6
            assert np.all(np.abs(got[k] - want) <= tol), (k, step, np.max(np.abs(got[k] - want) - tol))
        assert np.any(got["w1"] != wt["w1"])


def test_short_training_run_tracks_oracle(caps, tiny):
    """Five full-batch Adam steps on the GPU against the same five steps of
    the oracle (FP64 gradients with the GPU's BF16 operand roundings): the
    per-step losses agree within 1e-3 and the weight changes within 2% of
    their norm (a gradient entry near zero may differ in sign between FP32
    and FP64 accumulation, which moves that entry by up to 2 lr)."""
    w, ix = tiny
    rng = np.random.default_rng(5)
    dp = R.pad_width(w.d)
    wt = _weights(rng, 32, dp, 16)
    lr, b1, b2, eps = 2e-3, 0.9, 0.999, 1e-8
    labels = rng.integers(-1, 16, size=(w.n_q, 3)).astype(np.int32)
    ix.router_set(**wt, hidden=32, in_scale=0.5, in_shift=0.0)
    gpu_loss = ix.router_train(w.q, w.con_off, w.con_attr, w.con_val, labels, hidden=32, epochs=5, batch=w.n_q,
                               reset=0, lr=lr, beta1=b1, beta2=b2, eps=eps, in_scale=0.5, in_shift=0.0)
    x = R.input_rows(w.q, w.con_off, w.con_attr, w.con_val, w.dense_vocab, w.label_vocab, 0.5, 0.0)
    params = {k: v.astype(np.float64) for k, v in wt.items()}
    mom = {k: np.zeros_like(v) for k, v in params.items()}
    vel = {k: np.zeros_like(v) for k, v in params.items()}
    orc_loss = []
    for step in range(1, 6):
        f32 = {k: v.astype(np.float32) for k, v in params.items()}   # the GPU's masters are FP32
        loss, g = R.loss_and_grads(x, labels, **f32)
        orc_loss.append(loss)
        params = R.adam(params, g, mom, vel, step, lr, b1, b2, eps)
    assert np.allclose(gpu_loss, orc_loss, rtol=1e-3), (gpu_loss, orc_loss)
    got = ix.router_get()
    for k in params:
        assert _rel(got[k] - wt[k], params[k] - wt[k]) < 0.02, k


@pytest.mark.parametrize("b,hid,rows", [(13, 48, 77), (200, 144, 1), (1000, 80, 700), (136, 272, 1100)])
def test_gradient_shapes(caps, b, hid, rows):
    """The transposed products at their edges: output widths that are not
    multiples of 8 or of a tile, batches that are not multiples of 8, a single
    row, batches whose rows are split (more than 512)."""
    w = synth.make_tiny(960 + b, n=2000, d=20, n_q=rows, vocabs=(3, 4), b=b, h=1, cmin=0, cmax=2)
    ix = caps.Index.from_workload(w, kmeans_iters=1)
    rng = np.random.default_rng(b)
    wt = _weights(rng, hid, R.pad_width(w.d), b)
    ix.router_set(**wt, hidden=hid, in_scale=0.9, in_shift=0.1)
    labels = rng.integers(-1, b, size=(rows, 5)).astype(np.int32)
    labels[:, 3] = labels[:, 0]   # (a repeated label counts once)
    loss, g = ix.router_grads(w.q, w.con_off, w.con_attr, w.con_val, labels)
    x = R.input_rows(w.q, w.con_off, w.con_attr, w.con_val, w.dense_vocab, w.label_vocab, 0.9, 0.1)
    want_loss, want = R.loss_and_grads(x, labels, **wt)
    assert abs(loss - want_loss) <= 1e-4 * abs(want_loss)
    for k in ("w1", "b1", "w2", "b2"):
        assert _rel(g[k], want[k]) < 1e-4, k
    ix.close()
