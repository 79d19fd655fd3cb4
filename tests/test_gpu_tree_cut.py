"""Per-query tree searches with the library's own number of subtree searches
(16, 32 or 64 by tree and batch size), dealt by query or by subtree: batches and
trees on both sides of each choice, trees with leaves above the cut, fewer rows than k.  Results equal the
oracle's sequential search."""
import numpy as np
import pytest

import oracle
import synth

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n, nq, k", [(1, 3, 5), (40, 5, 64), (700, 9, 10), (19_999, 200, 64), (20_000, 200, 10),
                                      (33_000, 128, 64), (66_000, 64, 1), (66_000, 65, 10), (270_000, 130, 10),
                                      (530_000, 70, 20),
                                      (19_999, 600, 10), (20_000, 600, 64), (99_999, 600, 1), (100_000, 600, 1)])
def test_default_cut_matches_oracle(n, nq, k):
    import paper_2107_03368_amd as qd
    import torch
    db = synth.gen_db(n, 5000 + n)
    q, _ = synth.gen_queries(db, nq, 5001 + nq, 0.2, 0.6)
    q[0] = db[n // 2]
    t = lambda a: torch.from_numpy(np.ascontiguousarray(a).view(np.int64)).to("cuda:0")
    tree = qd.tree_build(t(db))
    rows = np.unique(np.linspace(0, nq - 1, 24).astype(int))
    ref = oracle.knn_brute(db, q[rows], k)
    for order in (qd.ORDER_BEST_FIRST, qd.ORDER_DEPTH_FIRST):
        got = [x.cpu().numpy()[rows] for x in qd.knn_tree(tree, t(q), k, order=order)[:4]]
        for a, b in zip(got, (ref.idx, ref.missed, ref.extra, ref.dist)):
            assert np.array_equal(a.view(b.dtype), b)
