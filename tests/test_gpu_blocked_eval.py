"""The blocked search's evaluation at the edges of its units: lists around 64
queries and their multiples, a last block with rows in one half only, one row
or a full half.  Results equal the oracle's sequential search."""
import numpy as np
import pytest

import oracle
import synth

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n", [20_224, 20_225, 20_352, 20_353])
@pytest.mark.parametrize("nq", [16, 63, 65, 128, 257, 600])
def test_units_match_oracle(n, nq):
    import paper_2107_03368_amd as qd
    import torch
    db = synth.gen_db(n, 6100 + n)
    q, _ = synth.gen_queries(db, nq, 6200 + nq, 0.2, 0.6)
    t = lambda a: torch.from_numpy(np.ascontiguousarray(a).view(np.int64)).to("cuda:0")
    tree = qd.tree_build(t(db))
    q[-1] = db[tree.export()["perm"][-1]]  # the last leaf-order row itself
    rows = np.unique(np.r_[np.linspace(0, nq - 1, 20).astype(int), nq - 1])
    for k in (1, 20):
        ref = oracle.knn_brute(db, q[rows], k)
        got = qd.knn_tree(tree, t(q), k, order=qd.ORDER_BLOCKED, schedule=(1, 0, 0))[:4]
        for a, b in zip(got, (ref.idx, ref.missed, ref.extra, ref.dist)):
            assert np.array_equal(a.cpu().numpy()[rows].view(b.dtype), b)
