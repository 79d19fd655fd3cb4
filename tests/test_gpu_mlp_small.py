"""Gradients of few pairs: their workspace, and as many chunks per query as the
pairs fill, against the oracle."""
import numpy as np
import pytest

import synth
from oracle import mlp as omlp
from small_pool import small_pool
from test_gpu_mlp_tiles import _case, _t

pytestmark = pytest.mark.gpu


# Partial sums for 64 chunks of every query: 2.6 MB and 17.6 MB.
@pytest.mark.parametrize("sizes,megabytes", [([10], 2), ([50] * 8, 6)])
def test_few_pairs_need_little_memory(sizes, megabytes):
    import torch
    import paper_2107_03368_amd as qd
    q, qoff, pq, feat, labels, params = _case(sizes, 3)
    model, args = qd.Model(_t(params)), [_t(a) for a in (q, qoff, pq, feat, labels)]
    g, loss = qd.model_gradients(model, *args)
    with small_pool(megabytes):
        g2, loss2 = qd.model_gradients(model, *args)
    assert torch.equal(g, g2) and torch.equal(loss, loss2)


# one query around the pairs of one, two and all 64 chunks; few and many queries of unlike sizes
@pytest.mark.parametrize("sizes", [[64], [127], [128], [129], [4_095], [4_097], [9_000], [0, 0, 700, 3], [70, 2_000] * 9],
                         ids=lambda s: f"{len(s)}q_{sum(s)}p")
def test_chunks_match_the_oracle(sizes):
    import paper_2107_03368_amd as qd
    q, qoff, pq, feat, labels, params = _case(sizes, 5)
    g, loss = qd.model_gradients(qd.Model(_t(params)), *(_t(a) for a in (q, qoff, pq, feat, labels)))
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
