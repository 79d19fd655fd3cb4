"""The frontier-order model's fused kernels at the edges of their 64-pair
tiles: scores and gradients for one pair, around 32 and 64 pairs, ragged and
empty query groups, and more pairs than one pass of the grid takes."""
import numpy as np
import pytest

import synth
from oracle import mlp as omlp

pytestmark = pytest.mark.gpu


def _case(sizes, seed):
    rng = np.random.default_rng(seed)
    sizes = np.asarray(sizes)
    db = synth.gen_db(len(sizes), 40 + seed)
    q, _ = synth.gen_queries(db, len(sizes), 50 + seed, 0.1, 0.5)
    qoff = np.concatenate([[0], np.cumsum(sizes)]).astype(np.int64)
    pq = np.repeat(np.arange(len(sizes), dtype=np.int32), sizes)
    feat = rng.random((len(pq), 32), dtype=np.float32)
    labels = (rng.random(len(pq)) < 0.3).astype(np.float32)
    params = synth.uniform_f32(omlp.NPARAMS, 60 + seed, -0.05, 0.05)
    return q, qoff, pq, feat, labels, params


def _t(a):
    import torch
    return torch.from_numpy(a.view(np.int64) if a.dtype == np.uint64 else a).to("cuda:0")


def _bf16(x):
    u = np.asarray(x, np.float32).view(np.uint32).astype(np.uint64)
    return ((((u + 0x7FFF + ((u >> 16) & 1)) >> 16) << 16).astype(np.uint32)).view(np.float32).astype(np.float64)


def _score_bound(params, q, pq, feat):
    """Derived: the layer-1 sums over up to 4096 + 33 terms and the layer-2 sums over 512 run in fp32 (relative
    error of a sum at most terms * 2^-24 of the sum of magnitudes, here over the terms present), and the layer-1
    activation is kept to 2^-17 as two bf16 terms.  Both reach the score through |W2| and |w3|."""
    o, parts = 0, []
    for _, shape in omlp.SIZES:
        n = int(np.prod(shape))
        parts.append(np.abs(_bf16(params[o:o + n]).reshape(shape)))
        o += n
    w1q, w1f, b1, w2, b2, w3, b3 = parts
    bits = np.unpackbits(q.view(np.uint8), bitorder="little").reshape(len(q), 4096).astype(np.float64)
    terms = bits.sum(1).max() + 33
    h1 = (bits @ w1q + b1)[pq] + np.abs(feat.astype(np.float64)) @ w1f
    h2 = h1 @ w2 + b2
    rel = terms * 2.0 ** -24 + 2.0 ** -17 + 512 * 2.0 ** -24 + 257 * 2.0 ** -24
    return rel * (h2 @ w3.reshape(-1) + np.abs(b3).sum())


SIZES = [[1], [31], [32], [33], [63, 1], [65], [64, 64], [0, 7, 0, 130, 1, 0, 95], [200] * 5 + [1] * 70, [5000] * 9]


@pytest.mark.parametrize("sizes", SIZES, ids=lambda s: f"{len(s)}q_{sum(s)}p")
def test_tiles_match_the_oracle(sizes):
    import torch
    import paper_2107_03368_amd as qd
    q, qoff, pq, feat, labels, params = _case(sizes, len(sizes))
    model = qd.Model(_t(params))
    s = qd.model_forward(model, _t(q), _t(pq), _t(feat)).cpu().numpy().astype(np.float64)
    ref, _ = omlp.forward(params, q, pq, feat)
    assert (np.abs(s - ref) <= _score_bound(params, q, pq, feat)).all()

    g, loss = qd.model_gradients(model, _t(q), _t(qoff), _t(pq), _t(feat), _t(labels))
    g2, loss2 = qd.model_gradients(model, _t(q), _t(qoff), _t(pq), _t(feat), _t(labels))
    assert torch.equal(g, g2) and torch.equal(loss, loss2)
    g = g.cpu().numpy().astype(np.float64)
    rloss, rg = omlp.loss_and_grad(params, q, pq, feat, labels)
    assert abs(loss.item() - rloss) <= 1e-4 * abs(rloss) + 1e-6
    o = 0
    for name, shape in omlp.SIZES:
        n = int(np.prod(shape))
        a, b = g[o:o + n], rg[o:o + n]
        o += n
        # d2 is rounded to bf16 (2^-9 of each entry); 1e-2 of the block covers it and the fp32 sums
        assert np.linalg.norm(a - b) <= 1e-2 * np.linalg.norm(b) + 1e-12, name


@pytest.mark.parametrize("nq,n_scored", [(1, 1), (3, 1), (70, 1), (40, 3), (9, 63), (5, 64), (4, 65), (3, 511)])
def test_scores_of_a_grid_of_pairs(nq, n_scored):
    import torch
    import paper_2107_03368_amd as qd
    db = synth.gen_db(20_000, 77)
    q, _ = synth.gen_queries(db, nq, 78, 0.1, 0.5)
    tree = qd.tree_build(_t(db))
    model = qd.Model(_t(synth.uniform_f32(omlp.NPARAMS, 79, -0.05, 0.05)))
    s = qd.model_score_tree(model, tree, _t(q), n_scored)
    pq = np.repeat(np.arange(nq, dtype=np.int32), n_scored)
    pn = np.tile(np.arange(n_scored, dtype=np.int32), nq)
    feat = qd.model_features(tree, _t(q), _t(pq), _t(pn))
    assert torch.equal(s.view(-1), qd.model_forward(model, _t(q), _t(pq), feat))
