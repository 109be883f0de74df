"""Workloads of the library as its users run them, for timing and comparing two builds.

Most cases are filtered searches: a batch of queries with attribute constraints
against a resident index, from one query to the 10k batch of the headline
benchmark, in every storage format, search mode and attribute kind.  One case
builds an index from host arrays and one trains the learned router.

  listed()            the named cases
  draw(rng)           one more case of the same ranges
  prepare(case, seed) corpus, index and queries (or host arrays), from the seed
  run(state)          one call as a program makes it
  exact(case, seed)   the floating outputs in 64 bits, with plain torch
  work(case)          bytes and operations one pass cannot do without
"""
import numpy as np
import torch

import paper_2308_15014_amd as caps

OR = -1   # separates the AND-terms of a disjunctive query

# Corpora: "ints": uniform integers 0..255, squared L2; "mixture": 16 Gaussian
# components, squared L2; "unit": unit Gaussians, inner product.
# Attributes: "dense": three single values (10/50/200, Zipf 1.0); "labels": sets
# of up to `per_point` labels of `label_vocab` (Zipf 1.1); "both".


def _search(name, **over):
    c = dict(name=name, what="search", corpus="ints", attrs="dense", n=1_000_000, d=128, b=1024, h=2,
             precision="bf16", nq=10_000, k=10, nprobe=624, mode=0, routing=0, disjunctive=False,
             counters=False, per_point=0, label_vocab=0)
    c.update(over)
    return c


def listed():
    return [
        # an interactive lookup: one query, few probes; latency alone counts
        _search("one query", nq=1, nprobe=64),
        # the small parity configuration: the FP32 index that a first-time user builds
        _search("10k x 32 fp32", corpus="mixture", n=10_000, d=32, b=32, precision="none", nq=100, nprobe=4),
        # the mean batch of the serving loop at 100k queries/s
        _search("serving batch of 24", nq=24),
        # a serving batch over dense values and labels, FP16 copy
        _search("serving batch of 200, labels", attrs="both", precision="fp16", h=4, nq=200, nprobe=576,
                per_point=8, label_vocab=5000),
        # the headline: 10k queries at recall@10 0.9
        _search("10k queries bf16"),
        # the same without a low-precision copy (the default of Index.build)
        _search("10k queries fp32", precision="none"),
        # precision mode with the learned router: approximate scan, exact rerank
        _search("10k queries routed rerank", mode=1, routing=1, nprobe=608),
        # angular corpus with label sets, FP8 copy, three quarters of the partitions
        _search("4k queries fp8 labels", corpus="unit", attrs="labels", d=96, h=4, precision="fp8", nq=4096,
                nprobe=768, per_point=8, label_vocab=1000),
        # the serving corpus's shape (dense values and labels, FP16), a full batch
        _search("8k queries fp16 labels", attrs="both", n=2_000_000, b=2048, h=4, precision="fp16", nq=8192,
                nprobe=1152, per_point=8, label_vocab=5000),
        # ragged sizes, OR constraints, a long result list
        _search("777 queries ragged", corpus="mixture", n=123_457, d=100, b=300, h=3, precision="none", nq=777, k=50,
                nprobe=75, disjunctive=True),
        # index build from host arrays, exported for a checkpoint
        dict(name="build 500k x 128", what="build", corpus="ints", attrs="dense", n=500_000, d=128, b=512, h=2,
             precision="bf16", iters=10, per_point=0, label_vocab=0),
        # one epoch of the learned router
        dict(name="train router", what="train", corpus="ints", attrs="dense", n=100_000, d=128, b=1024, h=2,
             precision="bf16", nq=100_000, hidden=1024, batch=4096, per_point=0, label_vocab=0),
    ]


def _log(rng, lo, hi):
    return int(round(lo * (hi / lo) ** rng.random()))


def draw(rng):
    u = rng.random()
    attrs = rng.choice(["dense", "dense", "labels", "both"])
    labels = attrs != "dense"
    case = dict(corpus=rng.choice(["ints", "mixture", "unit"]), attrs=attrs, d=rng.choice([32, 64, 96, 100, 128, 128, rng.randint(17, 256)]),
                h=rng.randint(0, 4), precision=rng.choice(["none", "bf16", "bf16", "fp16", "fp8"]),
                per_point=rng.choice([8, 8, 8, 24, 100]) if labels else 0,
                label_vocab=rng.choice([100, 1000, 5000]) if labels else 0)
    if u < 0.08:
        n = _log(rng, 10_000, 500_000)
        return dict(case, what="build", n=n, b=max(8, n // rng.randint(300, 1300)), iters=rng.randint(2, 10))
    if u < 0.16:
        return dict(case, what="train", attrs="dense", per_point=0, label_vocab=0, n=_log(rng, 10_000, 100_000), b=rng.choice([64, 256, 1000, 1024]),
                    nq=_log(rng, 2_000, 100_000), hidden=rng.choice([256, 512, 1024]), batch=rng.choice([1000, 2048, 4096]))
    n = _log(rng, 10_000, 1_000_000 if case["per_point"] <= 8 else 200_000)
    b = max(8, min(2048, n // rng.randint(300, 1300)))
    nq = _log(rng, 1, 10_000)
    nprobe = max(1, min(b, _log(rng, max(1, b // 100), b)))
    mode = rng.choice([0, 0, 0, 1, 2]) if case["precision"] != "none" else 0
    return dict(case, what="search", n=n, b=b, nq=nq, k=rng.choice([1, 10, 10, 10, 20, rng.randint(2, 64)]),
                nprobe=nprobe, mode=mode, routing=0, disjunctive=rng.random() < 0.15, counters=rng.random() < 0.15)


# ------------------------------------------------------------------ inputs
DENSE_VOCAB = [10, 50, 200]


def _generator(seed, stream, device="cuda"):
    return torch.Generator(device).manual_seed(int(seed) * 16 + stream)


def _zipf(shape, vocab, s, g):
    cdf = torch.cumsum(torch.arange(1, vocab + 1, dtype=torch.float64, device="cuda") ** -s, 0)
    u = torch.rand(shape, generator=g, device="cuda", dtype=torch.float64) * cdf[-1]
    return torch.searchsorted(cdf, u, right=True).clamp_(max=vocab - 1).to(torch.int32)


def _vectors(case, count, g, means):
    d = case["d"]
    if case["corpus"] == "ints":
        return torch.randint(0, 256, (count, d), generator=g, device="cuda", dtype=torch.int32).float()
    x = torch.randn((count, d), generator=g, device="cuda")
    if case["corpus"] == "unit":
        return x / x.norm(dim=1, keepdim=True)
    return x + means[torch.randint(0, means.shape[0], (count,), generator=g, device="cuda")]


def _corpus(case, seed):
    """Vectors [n, d], dense values [n, 3] or None, padded label sets [n, per_point] (ascending, -1 at the end) or None."""
    g = _generator(seed, 1)
    means = 2.0 * torch.randn((16, case["d"]), generator=g, device="cuda")
    x = _vectors(case, case["n"], g, means)
    dense = labels = None
    if case["attrs"] != "labels":
        dense = torch.stack([_zipf((case["n"],), v, 1.0, g) for v in DENSE_VOCAB], 1)
    if case["attrs"] != "dense":
        L, V = case["per_point"], case["label_vocab"]
        lab = _zipf((case["n"], L), V, 1.1, g)
        size = torch.randint(1, L + 1, (case["n"], 1), generator=g, device="cuda")
        lab[torch.arange(L, device="cuda")[None, :] >= size] = V
        lab = lab.sort(dim=1).values
        lab[:, 1:][lab[:, 1:] == lab[:, :-1]] = V   # a set holds a label once
        lab = lab.sort(dim=1).values
        labels = torch.where(lab == V, -1, lab)
    return x, dense, labels, means


def _frequency(case, dense, labels):
    """Share of points that hold each value of the slots a constraint is copied from."""
    f = []
    if dense is not None:
        f += [torch.bincount(dense[:, a].long(), minlength=v).double() / case["n"] for a, v in enumerate(DENSE_VOCAB)]
    if labels is not None:
        held = torch.bincount((labels + 1).flatten().long(), minlength=case["label_vocab"] + 1)[1:].double() / case["n"]
        f.append(held)
    return f


def _terms(case, count, cmax, g, dense, labels, freq):
    """`count` AND-terms of 1..cmax constraints copied from a random point each, redrawn while their share of points (as
    if independent) lies outside 0.05 % .. 40 %: (chosen [count, slots], attribute [slots], value [count, slots])."""
    nd = 0 if dense is None else dense.shape[1]
    slots = nd + (0 if labels is None else labels.shape[1])
    attr = torch.tensor(list(range(nd)) + [nd] * (slots - nd), device="cuda")
    pick = torch.zeros((count, slots), dtype=torch.bool, device="cuda")
    val = torch.zeros((count, slots), dtype=torch.int64, device="cuda")
    todo = torch.arange(count, device="cuda")
    for attempt in range(30):
        k = todo.numel()
        if k == 0:
            break
        p = torch.randint(0, case["n"], (k,), generator=g, device="cuda")
        v = torch.cat([t[p] for t in (dense, labels) if t is not None], 1).long()
        key = torch.rand((k, slots), generator=g, device="cuda")
        key[v < 0] = 2.0
        c = torch.randint(1, cmax + 1, (k, 1), generator=g, device="cuda")
        ch = (key.argsort(1).argsort(1) < c) & (v >= 0)
        share = torch.ones(k, dtype=torch.float64, device="cuda")
        for s in range(slots):
            share *= torch.where(ch[:, s], freq[min(s, nd)][v[:, s].clamp(min=0)], 1.0)
        ok = (share >= 5e-4) & (share <= 0.4) if attempt < 29 else torch.ones(k, dtype=torch.bool, device="cuda")
        pick[todo[ok]], val[todo[ok]] = ch[ok], v[ok]
        todo = todo[~ok]
    return pick, attr, val


def _constraints(case, nq, g, dense, labels):
    """Per query a list of AND-terms, each a list of (attribute, value), as CSR arrays with OR separators."""
    freq = _frequency(case, dense, labels)
    nt = np.ones(nq, np.int64)
    if case.get("disjunctive"):
        nt = torch.randint(1, 4, (nq,), generator=g, device="cuda").cpu().numpy()
    pick, attr, val = _terms(case, int(nt.sum()), 3 if case["attrs"] == "dense" else 4, g, dense, labels, freq)
    pick, attr, val = pick.cpu().numpy(), attr.cpu().numpy(), val.cpu().numpy()
    rows, cols = np.nonzero(pick)
    a, v = attr[cols], val[rows, cols]
    first = np.cumsum(nt) - nt                       # each query's first term
    sep = np.setdiff1d(np.arange(int(nt.sum())), first)   # terms after an OR
    order = np.argsort(np.concatenate([rows * 2 + 1, sep * 2]), kind="stable")
    a = np.concatenate([a, np.full(sep.size, OR)])[order]
    v = np.concatenate([v, np.zeros(sep.size, np.int64)])[order]
    per_term = np.bincount(rows, minlength=pick.shape[0])
    per_term[sep] += 1
    off = np.concatenate([[0], np.cumsum(np.add.reduceat(per_term, first))])
    return off.astype(np.int32), a.astype(np.int32), v.astype(np.int32)


def _init_ids(case, seed):
    return np.random.default_rng(seed).choice(case["n"], case["b"], replace=False).astype(np.int32)


def _host(case, x, dense, labels):
    """The host arrays Index.build takes."""
    kw = dict(x=x.cpu().numpy())
    if dense is not None:
        kw.update(dense=dense.cpu().numpy().astype(np.uint32), dense_vocab=DENSE_VOCAB)
    if labels is not None:
        held = labels >= 0
        off = torch.zeros(case["n"] + 1, dtype=torch.int64, device="cuda")
        off[1:] = held.sum(1).cumsum(0)
        kw.update(label_off=off.cpu().numpy(), labels=labels[held].cpu().numpy().astype(np.uint32), label_vocab=case["label_vocab"])
    return kw


def _metric(case):
    return 1 if case["corpus"] == "unit" else 0


def _build(case, seed, host):
    return caps.Index.build(**host, metric=_metric(case), n_partitions=case["b"], kmeans_iters=case.get("iters", 10), aft_height=case["h"],
                            init_ids=_init_ids(case, seed), precision=case["precision"])


def _queries(case, seed, means, dense, labels, nq, stream):
    g = _generator(seed, stream)
    q = _vectors(case, nq, g, means)
    return (q, *(torch.from_numpy(t).cuda() for t in _constraints(case, nq, g, dense, labels)))


def prepare(case, seed):
    x, dense, labels, means = _corpus(case, seed)
    host = _host(case, x, dense, labels)
    if case["what"] == "build":
        return dict(case=case, seed=seed, host=host)
    ix = _build(case, seed, host)
    q = _queries(case, seed, means, dense, labels, case["nq"], 2)
    if case["what"] == "train":
        # labels as a program makes them: the partitions of each query's filtered nearest neighbours
        near = ix.search(*q, 10, min(case["b"], 64))[0]
        return dict(case=case, ix=ix, q=q, labels=ix.router_labels(near))
    if case["routing"]:
        t = _queries(case, seed, means, dense, labels, 20_000, 3)
        near = ix.search(*t, 10, case["nprobe"])[0]
        ix.router_train(*t, ix.router_labels(near), hidden=1024, epochs=1, batch=2000, lr=1e-3, in_scale=1 / 128, in_shift=-1.0, seed=seed)
    return dict(case=case, ix=ix, q=q)


# ------------------------------------------------------------------ one pass
def run(state):
    c = state["case"]
    if c["what"] == "build":
        ix = _build(c, state["seed"], state["host"])
        out = ix.export()
        ix.close()
        return out
    if c["what"] == "train":
        loss = state["ix"].router_train(*state["q"], state["labels"], hidden=c["hidden"], epochs=1, batch=c["batch"], lr=1e-3,
                                        in_scale=1 / 128, in_shift=-1.0, seed=1)
        return dict(state["ix"].router_get(), loss=loss)
    return list(state["ix"].search(*state["q"], c["k"], c["nprobe"], mode=c["mode"], routing=c["routing"], disjunctive=c["disjunctive"],
                                   counters=c["counters"]))


# ------------------------------------------------------------------ 64 bits
def _scores(case, x, c):
    return -(x @ c.T) if _metric(case) else (c * c).sum(1)[None, :] - 2.0 * (x @ c.T)


def _lloyd(case, x, seed):
    """Centroids and assignment of seeded Lloyd k-means in 64 bits."""
    n, b = case["n"], case["b"]
    cent = x[torch.from_numpy(_init_ids(case, seed)).cuda().long()].clone()
    for it in range(case.get("iters", 10) + 1):
        a = torch.cat([_scores(case, x[i:i + 65536], cent).argmin(1) for i in range(0, n, 65536)])
        if it == case.get("iters", 10):
            return cent, a
        size = torch.bincount(a, minlength=b)
        s = torch.zeros_like(cent).index_add_(0, a, x) / size.clamp(min=1)[:, None]
        if _metric(case):
            s = s / s.norm(dim=1, keepdim=True).clamp(min=1e-300)
        cent = torch.where((size > 0)[:, None], s, cent)


def exact(case, seed):
    if case["what"] == "train" or case.get("routing"):
        return None   # the weights start from the library's own random values
    x32, dense, labels, means = _corpus(case, seed)
    x = x32.double()
    cent, assign = _lloyd(case, x, seed)
    if case["what"] == "build":
        return dict(centroids=cent, assign=None, level=None, perm=None, offs=None, tags=None)
    q, off, attr, val = _queries(case, seed, means, dense, labels, case["nq"], 2)
    q, off, attr, val = q.double(), off.tolist(), attr.tolist(), val.tolist()
    nd = 0 if dense is None else dense.shape[1]
    k, n, ip = case["k"], case["n"], _metric(case)
    xx = (x * x).sum(1)
    out = []
    step = max(1, min(256, (1 << 28) // n))
    for i in range(0, case["nq"], step):
        qs = q[i:i + step]
        probed = torch.zeros((qs.shape[0], case["b"]), dtype=torch.bool, device="cuda")
        probed.scatter_(1, _scores(case, qs, cent).topk(case["nprobe"], dim=1, largest=False).indices, True)
        dist = -(qs @ x.T) if ip else (qs * qs).sum(1)[:, None] + xx[None, :] - 2.0 * (qs @ x.T)
        valid = probed[:, assign]
        for r in range(qs.shape[0]):
            some = torch.zeros(n, dtype=torch.bool, device="cuda")
            term = torch.ones(n, dtype=torch.bool, device="cuda")
            for e in range(off[i + r], off[i + r + 1]):
                if attr[e] == OR:
                    some |= term
                    term = torch.ones(n, dtype=torch.bool, device="cuda")
                else:
                    term &= dense[:, attr[e]] == val[e] if attr[e] < nd else (labels == val[e]).any(1)
            valid[r] &= some | term
        dist.masked_fill_(~valid, float("inf"))
        best = dist.topk(min(k, n), dim=1, largest=False).values
        out.append(-best if ip else best)
    return [None, torch.cat(out)] + [None] * (2 if case["counters"] else 0)


# ------------------------------------------------------------------ what a pass needs
def work(case):
    n, d, b = case["n"], case["d"], case["b"]
    attr = (4 if case["attrs"] != "labels" else 0) + (case["per_point"] + 1)   # packed values; two bytes for each label held
    attr = attr if case["attrs"] != "dense" else 4
    if case["what"] == "build":
        it = case["iters"]
        low = {"none": 0, "bf16": 2, "fp16": 2, "fp8": 1}[case["precision"]]
        return dict(bytes=n * (d * (8 + low) + 2 * attr + 13), flops=2.0 * n * b * d * (it + 1) + n * d * it)
    if case["what"] == "train":
        w = case["hidden"] * (d + 64 + b)
        steps = -(-case["nq"] // case["batch"])
        return dict(bytes=case["nq"] * (4 * d + 64) + steps * 24 * w, flops=6.0 * case["nq"] * w)
    # about 5 % of the points pass a query's filter (an OR of terms: 10 %)
    nq, f, sel = case["nq"], case["nprobe"] / b, 0.10 if case["disjunctive"] else 0.05
    cand = n * (1.0 - (1.0 - f) ** nq)
    surv = n * (1.0 - (1.0 - f * sel) ** nq)
    return dict(bytes=cand * attr + surv * 4 * d + b * 4 * d + nq * (4 * d + 8 * case["k"] + 24),
                flops=3.0 * d * nq * n * f * sel + 2.0 * nq * b * d)
