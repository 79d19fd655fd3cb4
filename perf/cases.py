"""Performance cases: the work a program has this library do, over its real range.

Each case is one pass through the public entry points of the Python package on
synthetic 64x64-bit descriptors: ring arcs of 2-8% density as database rows,
partial noisy copies of rows as queries (bits cleared with a probability drawn
per query, 8 bits flipped).  All inputs are drawn on the GPU from the seed.

Kinds
  scan     sequential search (knn_bruteforce), from one query over 10,000 rows
           to a batch of thousands
  planes   small batches over a bit-plane index built beforehand
  tree     the per-query tree search (best-first, the default order, or
           depth-first) on a tree built beforehand
  blocked  the batched tree search on the matrix cores
  build    index and search: the tree of a database, then one batch on it
  scores   object-level scores and the ranking of every query object
  plan     partial-object retrieval by votes through a captured plan
  learned  node scores of the frontier-order model, then the depth-first
           search they order
  train    the model's gradient over one batch of training pairs
"""
import functools
import math

import torch

import paper_2107_03368_amd as qd

BITS = 4096
DEV = "cuda"


def listed():
    return [
        # one descriptor against a small database: launches and latency
        dict(name="scan_10k_1q_k1", kind="scan", n=10_000, nq=1, k=1),
        # interactive batches over a large database: one pass over the rows
        dict(name="scan_10m_8q_k10", kind="scan", n=10_000_000, nq=8, k=10),
        # a small serving batch over the same database
        dict(name="scan_10m_64q_k10", kind="scan", n=10_000_000, nq=64, k=10),
        # a whole batch of queries, sequential search
        dict(name="scan_1m_4096q_k10", kind="scan", n=1_000_000, nq=4096, k=10),
        # small batches where an index was built for them
        dict(name="planes_10m_16q_k10", kind="planes", n=10_000_000, nq=16, k=10),
        # the default tree search, query by query, ragged sizes
        dict(name="tree_1m_509q_k10", kind="tree", order="best", n=1_000_003, nq=509, k=10),
        # the largest: the batched tree search of the benchmark's workload
        dict(name="blocked_10m_8192q_k10", kind="blocked", n=10_000_000, nq=8192, k=10),
        # a database arrives, is indexed and answers its first batch
        dict(name="build_1m_256q_k10", kind="build", n=1_000_000, nq=256, k=10),
        # object matching: ragged query objects against every database object
        dict(name="scores_300x5000_32qo", kind="scores", n_obj=300, per_obj=5000, nqo=32, mmin=50, mmax=800),
        # retrieval of a serving batch of query objects through a plan
        dict(name="plan_300x5000_48qo_k5", kind="plan", n_obj=300, per_obj=5000, nqo=48, mmin=50, mmax=300, k=5),
        # the learned order's inference and the search it leads
        dict(name="learned_1m_512q_k10", kind="learned", n=1_000_000, nq=512, k=10, n_scored=2047),
        # one optimizer step's gradient of the order model
        dict(name="train_256q_1201p", kind="train", nq=256, per_q=1201),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["scan", "scan", "planes", "tree", "blocked", "build", "scores", "plan", "learned", "train"])
    k = rng.choice([1, 1, 5, 10, 10, 10, 50])
    if kind == "scan":
        n = _log_int(rng, 1_000, 10_000_000)
        return dict(kind=kind, n=n, nq=_log_int(rng, 1, max(1, min(8192, 20_000_000_000 // n))), k=k)
    if kind == "planes":
        return dict(kind=kind, n=_log_int(rng, 10_000, 10_000_000), nq=_log_int(rng, 1, 64), k=k)
    if kind == "tree":
        return dict(kind=kind, order=rng.choice(["best", "depth"]), n=_log_int(rng, 10_000, 1_500_000),
                    nq=_log_int(rng, 1, 600), k=k)
    if kind == "blocked":
        n = _log_int(rng, 20_000, 10_000_000)
        return dict(kind=kind, n=n, nq=_log_int(rng, 64, 8192), k=k)
    if kind == "build":
        return dict(kind=kind, n=_log_int(rng, 20_000, 2_000_000), nq=_log_int(rng, 1, 1024), k=k)
    if kind == "scores":
        return dict(kind=kind, n_obj=_log_int(rng, 10, 400), per_obj=_log_int(rng, 300, 5_000),
                    nqo=_log_int(rng, 1, 48), mmin=20, mmax=_log_int(rng, 40, 800))
    if kind == "plan":
        return dict(kind=kind, n_obj=_log_int(rng, 20, 400), per_obj=_log_int(rng, 500, 5_000),
                    nqo=_log_int(rng, 1, 64), mmin=20, mmax=_log_int(rng, 40, 400), k=rng.choice([1, 5, 10]))
    if kind == "learned":
        return dict(kind=kind, n=_log_int(rng, 70_000, 1_500_000), nq=_log_int(rng, 1, 600), k=k,
                    n_scored=rng.choice([511, 1001, 2047]))
    return dict(kind="train", nq=_log_int(rng, 8, 512), per_q=_log_int(rng, 50, 2_000))


# ---- inputs -----------------------------------------------------------------


def _gen(seed, salt):
    return torch.Generator(device=DEV).manual_seed(seed * 1_000_003 + salt)


def _pack(bits):
    """(n, 4096) truth values -> (n, 64) int64 words, bit c of word r = column c of row r."""
    sh = torch.arange(64, device=bits.device, dtype=torch.int64)
    return (bits.view(-1, 64, 64).to(torch.int64) << sh).sum(-1)


def _unpack(rows, dtype):
    """(n, 64) int64 words -> (n, 4096) of 0 / 1."""
    sh = torch.arange(64, device=rows.device, dtype=torch.int64)
    return ((rows.unsqueeze(-1) >> sh) & 1).view(-1, BITS).to(dtype)


@functools.lru_cache(maxsize=1)
def _arcs():
    """A library of one-pixel ring arcs around the image centre: (words, pixels of each); the last is empty."""
    y, x = torch.meshgrid(torch.arange(64, device=DEV) - 31.5, torch.arange(64, device=DEV) - 31.5, indexing="ij")
    rad, ang = torch.sqrt(x * x + y * y).view(1, -1), torch.atan2(y, x).view(1, -1)
    start = (torch.arange(64, device=DEV) * (2 * math.pi / 64)).view(-1, 1, 1)
    length = (math.pi / 4 + torch.arange(29, device=DEV) * (7 * math.pi / 4 / 28)).view(1, -1, 1)
    sector = (torch.remainder(ang.view(1, 1, -1) - start, 2 * math.pi) <= length).view(-1, BITS)
    words, pops = [], []
    for i in range(59):
        arc = sector & ((rad - (2.0 + 0.5 * i)).abs() < 0.5)
        words.append(_pack(arc))
        pops.append(arc.sum(1))
    words.append(torch.zeros(1, 64, dtype=torch.int64, device=DEV))
    pops.append(torch.zeros(1, dtype=torch.int64, device=DEV))
    return torch.cat(words), torch.cat(pops)


def _rows(n, seed):
    """n database rows: 3 to 12 arcs, at most 327 pixels, more arcs while there are fewer than 82."""
    words, pops = _arcs()
    empty = words.shape[0] - 1
    out = torch.empty(n, 64, dtype=torch.int64, device=DEV)
    g = _gen(seed, 1)
    for r0 in range(0, n, 1 << 20):
        m = min(1 << 20, n - r0)
        want = torch.randint(3, 13, (m,), generator=g, device=DEV)
        total = torch.zeros(m, dtype=torch.int64, device=DEV)
        acc = out[r0:r0 + m]
        acc.zero_()
        for i in range(14):
            a = torch.randint(0, empty, (m,), generator=g, device=DEV)
            c = pops[a]
            take = ((want > i) | (total < 82)) & (total + c <= 327)
            acc |= words[torch.where(take, a, empty)]
            total += torch.where(take, c, 0)
    return out


def _partial(rows, seed, pmin, pmax):
    """Partial noisy copies of the given rows."""
    out = torch.empty_like(rows)
    g = _gen(seed, 2)
    for r0 in range(0, rows.shape[0], 8192):
        src = rows[r0:r0 + 8192]
        m = src.shape[0]
        p = pmin + (pmax - pmin) * torch.rand(m, 1, generator=g, device=DEV)
        keep = torch.rand(m, BITS, generator=g, device=DEV) >= p
        flip = torch.zeros(m, BITS, dtype=torch.bool, device=DEV)
        flip.scatter_(1, torch.randint(0, BITS, (m, 8), generator=g, device=DEV), True)
        out[r0:r0 + m] = (src & _pack(keep)) ^ _pack(flip)
    return out


def _queries(db, nq, seed, pmin=0.1, pmax=0.6):
    src = torch.randint(0, db.shape[0], (nq,), generator=_gen(seed, 3), device=DEV)
    return _partial(db[src], seed, pmin, pmax)


def _objects(case, seed):
    """Database rows by object, and query objects: random distinct rows of one object each, in random order."""
    n_obj, per = case["n_obj"], case["per_obj"]
    db = _rows(n_obj * per, seed)
    obj_of = (torch.arange(n_obj * per, device=DEV) // per).to(torch.int16)
    g = torch.Generator().manual_seed(seed * 1_000_003 + 4)
    sizes = torch.randint(case["mmin"], min(case["mmax"], per) + 1, (case["nqo"],), generator=g)
    src = torch.randint(0, n_obj, (case["nqo"],), generator=g)
    rows = torch.cat([o * per + torch.randperm(per, generator=g)[:m] for o, m in zip(src.tolist(), sizes.tolist())])
    off = torch.zeros(case["nqo"] + 1, dtype=torch.int64)
    off[1:] = sizes.cumsum(0)
    q = _partial(db[rows.to(DEV)], seed, 0.2, 0.7)
    return db, obj_of, q, off.to(DEV)


def _params(seed):
    """Model parameters as a fresh training starts from: uniform, scaled by the layer's inputs."""
    h = qd.MLP_HIDDEN
    g = _gen(seed, 5)

    def u(count, fan):
        return (torch.rand(count, generator=g, device=DEV) * 2 - 1) / math.sqrt(fan)

    return torch.cat([u(BITS * h, 256), u(qd.MLP_FEATURES * h, 32), u(h, 32), u(h * h, h), u(h, h), u(h, h), u(1, h)])


def _pairs(case, seed):
    """Training pairs grouped by query (ragged groups), their node features and labels."""
    g = _gen(seed, 6)
    nq, per = case["nq"], case["per_q"]
    sizes = torch.randint(max(1, per // 2), per + per // 2 + 1, (nq,), generator=g, device=DEV)
    qoff = torch.zeros(nq + 1, dtype=torch.int64, device=DEV)
    qoff[1:] = sizes.cumsum(0)
    pair_q = torch.repeat_interleave(torch.arange(nq, device=DEV, dtype=torch.int32), sizes)
    np_ = pair_q.shape[0]
    # shares of the query's bits a node misses, overall and by band, and the node's own terms
    miss = torch.rand(np_, 1, generator=g, device=DEV) * 0.6
    band = torch.rand(np_, 11, generator=g, device=DEV)
    band = band / band.sum(1, keepdim=True)
    own = torch.rand(np_, 8, generator=g, device=DEV)
    feat = torch.cat([miss, 1 - miss, own, miss * band, (1 - miss) * band], dim=1)
    feat[:, 6:8] = (feat[:, 6:8] < 0.5).float()
    labels = (torch.rand(np_, generator=g, device=DEV) < 0.25 * (0.6 - miss[:, 0]) / 0.6).float()
    return qoff, pair_q, feat.contiguous(), labels


def prepare(case, seed):
    kind = case["kind"]
    if kind in ("scores", "plan"):
        db, obj_of, q, off = _objects(case, seed)
        st = dict(case=case, db=db, obj_of=obj_of, q=q, off=off)
        if kind == "plan":
            st["tree"] = qd.tree_build(db)
            st["plan"] = qd.Plan(obj_of, case["n_obj"], case["nqo"] * case["mmax"], case["nqo"], case["k"],
                                 tree=st["tree"], order=qd.ORDER_BLOCKED)
    elif kind == "train":
        # queries alone: the pairs' features stand for their nodes
        q = _partial(_rows(case["nq"], seed), seed, 0.1, 0.6)
        qoff, pair_q, feat, labels = _pairs(case, seed)
        st = dict(case=case, q=q, qoff=qoff, pair_q=pair_q, feat=feat, labels=labels, model=qd.Model(_params(seed)))
    else:
        db = _rows(case["n"], seed)
        st = dict(case=case, db=db, q=_queries(db, case["nq"], seed))
        if kind == "planes":
            st["planes"] = qd.Planes(db)
        if kind in ("tree", "blocked", "learned"):
            st["tree"] = qd.tree_build(db)
        if kind == "learned":
            st["model"] = qd.Model(_params(seed))
    torch.cuda.synchronize()
    return st


def run(st):
    c = st["case"]
    kind = c["kind"]
    if kind == "scan":
        return qd.knn_bruteforce(st["db"], st["q"], c["k"])
    if kind == "planes":
        return qd.knn_planes(st["planes"], st["q"], c["k"])
    if kind == "tree":
        return qd.knn_tree(st["tree"], st["q"], c["k"],
                           order=qd.ORDER_BEST_FIRST if c["order"] == "best" else qd.ORDER_DEPTH_FIRST)
    if kind == "blocked":
        return qd.knn_tree(st["tree"], st["q"], c["k"], order=qd.ORDER_BLOCKED)
    if kind == "build":
        tree = qd.tree_build(st["db"])
        return qd.knn_tree(tree, st["q"], c["k"], order=qd.ORDER_BLOCKED)
    if kind == "scores":
        scores = qd.object_scores(st["db"], st["obj_of"], c["n_obj"], st["q"], st["off"])
        return scores, qd.score_rows(scores, normalize=False)
    if kind == "plan":
        return st["plan"].run(st["q"], st["off"])
    if kind == "learned":
        scores = qd.model_score_tree(st["model"], st["tree"], st["q"], c["n_scored"])
        return (scores,) + qd.knn_tree(st["tree"], st["q"], c["k"], order=qd.ORDER_DEPTH_FIRST, scores=scores)
    return qd.model_gradients(st["model"], st["q"], st["qoff"], st["pair_q"], st["feat"], st["labels"])


def work(case):
    """Bytes and operations the answer itself needs.  A (query, row) overlap is 4096 multiply-adds of bits.  The
    tree searches need at least every query against every 256-row block's summary and k blocks' rows."""
    kind, row = case["kind"], 512
    if kind == "train":
        pairs, h = case["nq"] * case["per_q"], qd.MLP_HIDDEN
        layers = qd.MLP_FEATURES * h + h * h + h
        # forward, then the two products of every layer backwards; the query layer once per set bit (about 170)
        flops = 6 * pairs * layers + 4 * case["nq"] * 170 * h
        return dict(bytes=pairs * (4 * qd.MLP_FEATURES + 8) + case["nq"] * row + 8 * qd.MLP_NPARAMS, flops=flops)
    if kind in ("scores", "plan"):
        n, nq = case["n_obj"] * case["per_obj"], case["nqo"] * (case["mmin"] + case["mmax"]) // 2
        if kind == "scores":
            return dict(bytes=(n + nq) * row + 8 * case["nqo"] * case["n_obj"], flops=2 * BITS * n * nq)
        return dict(bytes=(n + nq) * row + 4 * case["nqo"] * case["n_obj"], flops=2 * BITS * nq * (n // 256 + 256))
    n, nq, k = case["n"], case["nq"], case["k"]
    out = nq * k * 16
    if kind == "scan":
        return dict(bytes=(n + nq) * row + out, flops=2 * BITS * n * nq)
    if kind == "planes":
        return dict(bytes=min(nq * 170, BITS) * (n // 8) + nq * row + out, flops=2 * nq * 170 * n)
    search = 2 * BITS * nq * (n // 256 + 256)
    if kind == "blocked":
        return dict(bytes=(n + nq) * row + out, flops=search)
    if kind == "build":  # the rows in, their leaf order and images out
        return dict(bytes=2 * n * row + n * row // 16 + nq * row + out, flops=search)
    flops, bytes_ = 2 * BITS * nq * (n // 256), n // 32 * row + nq * (256 * row + row) + out
    if kind == "learned":
        h = qd.MLP_HIDDEN
        pairs = nq * case["n_scored"]
        flops += 2 * pairs * (qd.MLP_FEATURES * h + h * h + h) + 2 * nq * 170 * h
        bytes_ += pairs * 4 + case["n_scored"] * row + 4 * qd.MLP_NPARAMS
    return dict(bytes=bytes_, flops=flops)


# ---- the answers in 64 bits -----------------------------------------------------


def _exact_knn(db, q, k):
    """Distances of the k nearest rows by (key, row), as float64; short answers are padded with infinity."""
    qb = _unpack(q, torch.float32)
    pq = qb.sum(1).to(torch.int64)
    wa, wb = pq.clamp(min=1).view(-1, 1), (BITS - pq).clamp(min=1).view(-1, 1)
    best = torch.empty(q.shape[0], 0, dtype=torch.int64, device=DEV)
    step = max(256, min(1 << 17, (1 << 28) // max(1, q.shape[0])))
    for r0 in range(0, db.shape[0], step):
        tb = _unpack(db[r0:r0 + step], torch.float32)
        c = (qb @ tb.t()).to(torch.int64)  # counts up to 4096: exact
        key = (pq.view(-1, 1) - c) * wb + (tb.sum(1).to(torch.int64).view(1, -1) - c) * wa
        key = key << 32 | torch.arange(r0, r0 + tb.shape[0], device=DEV)
        best = torch.cat([best, key.topk(min(k, key.shape[1]), dim=1, largest=False).values], dim=1)
        best = best.topk(min(k, best.shape[1]), dim=1, largest=False, sorted=True).values
    dist = torch.full((q.shape[0], k), math.inf, dtype=torch.float64, device=DEV)
    dist[:, :best.shape[1]] = (best >> 32).double() / (wa * wb).double()
    return dist


def _exact_scores(st, c):
    """Sum over each query object's descriptors of the distance to the nearest row of every object."""
    db, q, off = st["db"], st["q"], st["off"].tolist()
    qb = _unpack(q, torch.float32)
    pq = qb.sum(1).to(torch.int64)
    wa, wb = pq.clamp(min=1).view(-1, 1), (BITS - pq).clamp(min=1).view(-1, 1)
    near = torch.empty(q.shape[0], c["n_obj"], dtype=torch.float64, device=DEV)
    for o in range(c["n_obj"]):
        tb = _unpack(db[o * c["per_obj"]:(o + 1) * c["per_obj"]], torch.float32)
        cnt = (qb @ tb.t()).to(torch.int64)
        key = (pq.view(-1, 1) - cnt) * wb + (tb.sum(1).to(torch.int64).view(1, -1) - cnt) * wa
        near[:, o] = key.amin(1).double() / (wa * wb).double().view(-1)
    return torch.stack([near[a:b].sum(0) for a, b in zip(off, off[1:])])


def _layers(seed):
    """The parameters, rounded to bf16 as the model computes with, in float64."""
    p = _params(seed).to(torch.bfloat16).double()
    h, f, out, at = qd.MLP_HIDDEN, qd.MLP_FEATURES, [], 0
    for shape in ((BITS, h), (f, h), (h,), (h, h), (h,), (h,), (1,)):
        size = math.prod(shape)
        out.append(p[at:at + size].view(shape))
        at += size
    return out


def _exact_gradients(st, seed):
    w1q, w1f, b1, w2, b2, w3, b3 = _layers(seed)
    qb, feat, y = _unpack(st["q"], torch.float64), st["feat"].double(), st["labels"].double()
    pq = st["pair_q"].long()
    n = feat.shape[0]
    u = qb @ w1q + b1
    h1 = (u[pq] + feat @ w1f).relu()
    h2 = (h1 @ w2 + b2).relu()
    s = h2 @ w3 + b3
    loss = (torch.nn.functional.softplus(s) - y * s).mean()
    ds = (torch.sigmoid(s) - y) / n
    d2 = ds.view(-1, 1) * w3 * (h2 > 0)
    d1 = (d2 @ w2.t()) * (h1 > 0)
    du = torch.zeros(qb.shape[0], d1.shape[1], dtype=torch.float64, device=DEV).index_add_(0, pq, d1)
    grads = [qb.t() @ du, feat.t() @ d1, d1.sum(0), h1.t() @ d2, d2.sum(0), h2.t() @ ds, ds.sum()]
    return torch.cat([g.reshape(-1) for g in grads]), loss.view(1)


def exact(case, seed):
    kind = case["kind"]
    if kind == "train":
        q = _partial(_rows(case["nq"], seed), seed, 0.1, 0.6)
        qoff, pair_q, feat, labels = _pairs(case, seed)
        return _exact_gradients(dict(q=q, pair_q=pair_q, feat=feat, labels=labels), seed)
    if kind == "plan":
        return None  # votes, winners and counts: whole numbers
    if kind == "scores":
        db, _, q, off = _objects(case, seed)
        return _exact_scores(dict(db=db, q=q, off=off), case), None
    if case["n"] * case["nq"] > 6_000_000_000:  # the products alone take too long
        return None
    db = _rows(case["n"], seed)
    q = _queries(db, case["nq"], seed)
    dist = _exact_knn(db, q, case["k"])
    if kind == "learned":
        return None, None, None, None, dist  # the scores' node features come from the library's own tree
    return None, None, None, dist
