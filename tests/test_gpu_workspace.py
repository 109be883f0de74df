"""The least workspace: a caller's array or a server's budget that holds one
query under the layout with 512 deferred pairs (exact search) or none
(approximate), and no copy or tables of small batches, is accepted, and the
results are those of an unbounded search."""
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
    # prec, d, label_vocab, mode, k, m, bytes of one query's layout at b = 40, h = 2
    ("none", 40, 0, 0, 10, 6, 6160),
    ("bf16", 40, 0, 0, 10, 6, 12816),
    ("bf16", 40, 0, 1, 10, 40, 19472),
    ("fp8", 40, 5, 0, 40, 40, 25104),
    ("fp8", 40, 5, 1, 10, 40, 19472),
    ("bf16", 200, 0, 0, 40, 6, 14608),
]


@pytest.mark.parametrize("case", CASES)
def test_one_query_fits(caps, case):
    prec, d, lv, mode, k, m, size = case
    w = synth.make_tiny(1400, n=3000, d=d, n_q=40, vocabs=(3,), label_vocab=lv, b=40, h=2, cmin=0, cmax=1)
    ix = caps.Index.from_workload(w, kmeans_iters=1, precision=prec)
    args = (w.q, w.con_off, w.con_attr, w.con_val, k, m)
    want = [t.cpu().numpy() for t in ix.search(*args, mode=mode)]
    one = [t.cpu().numpy() for t in ix.search_static(w.q[:1], w.con_off[:2], w.con_attr, w.con_val, k, m, mode=mode,
                                                     workspace_bytes=size)]
    assert np.array_equal(one[0], want[0][:1]) and np.array_equal(one[1], want[1][:1])
    more = [t.cpu().numpy() for t in ix.search_static(*args, mode=mode, workspace_bytes=3 * size)]   # (in sub-batches)
    assert np.array_equal(more[0], want[0]) and np.array_equal(more[1], want[1])
    srv = caps.Server(ix, k=k, nprobe=m, mode=mode, streams=2, workspace_bytes=size)
    try:
        assert srv.stats()["max_batch"] == 1
        tick = {srv.submit(w.q[i], w.con_attr[w.con_off[i]:w.con_off[i + 1]], w.con_val[w.con_off[i]:w.con_off[i + 1]]): i
                for i in range(w.n_q)}
        srv.drain(30)
        r = srv.poll(100)
        rows = [tick[t] for t in np.asarray(r["tickets"]).tolist()]
        assert sorted(rows) == list(range(w.n_q))
        assert np.array_equal(r["ids"], want[0][rows]) and np.array_equal(r["dist"], want[1][rows])
    finally:
        srv.close()
    ix.close()


def test_copy_gives_way_to_a_query(caps):
    """n = 20,000, b = m = 8192, k = 64: a copy of the rows (1.5 MB) and one
    query (4.7 MB) do not both fit 5 MiB.  Whether the batch is accepted does not
    depend on its size, above the copy's rule or below."""
    w = synth.make_tiny(1401, n=20_000, d=32, n_q=1700, vocabs=(3,), b=8192, h=2, cmin=0, cmax=1)
    ix = caps.Index.from_workload(w, kmeans_iters=0)
    args = (w.q, w.con_off, w.con_attr, w.con_val, 64, 8192)
    assert ix.workspace_bytes(1700, 64, 8192) > ix.workspace_bytes(1700, 64, 8192, mode=2)   # (a copy)
    want = [t.cpu().numpy() for t in ix.search(*args)]
    for n in (100, 1700):
        got = ix.search_static(w.q[:n], w.con_off[:n + 1], w.con_attr, w.con_val, 64, 8192, workspace_bytes=5 << 20)
        assert np.array_equal(got[0].cpu().numpy(), want[0][:n]) and np.array_equal(got[1].cpu().numpy(), want[1][:n])
    ix.close()
