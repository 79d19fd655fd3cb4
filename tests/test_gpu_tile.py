"""The 256 x 256 overlap tile and its pass test where they can go wrong: rows
and queries of every density from empty to full (the test's bound changes
with |q| and |t|), many rows tied at the k-th key, and row and query counts
one off the tile's multiples, on the sequential and the blocked search."""
import numpy as np
import pytest

import oracle
import synth

pytestmark = pytest.mark.gpu


def _dense(n, seed, counts):
    """Rows with exactly the given popcounts, repeated in turn, at random positions."""
    rng = np.random.default_rng(seed)
    bits = np.zeros((n, 4096), np.uint8)
    for i in range(n):
        bits[i, rng.permutation(4096)[:counts[i % len(counts)]]] = 1
    return np.packbits(bits, axis=1, bitorder="little").view(np.uint64)


def _t(a):
    import torch
    return torch.from_numpy(np.ascontiguousarray(a).view(np.int64)).to("cuda:0")


@pytest.mark.parametrize("n,nq,k", [(65_536, 160, 1), (65_537, 257, 10), (65_791, 255, 64), (66_048, 513, 10)])
def test_tile_at_every_density(n, nq, k):
    import paper_2107_03368_amd as qd
    counts = [0, 1, 2, 63, 170, 300, 2047, 2048, 2049, 4000, 4094, 4095, 4096]
    db = synth.gen_db(n, 900 + n)
    db[::97] = _dense(len(db[::97]), n, counts)
    db[5::50] = db[5]  # 1,300 tied rows
    q, _ = synth.gen_queries(db, nq, 901 + n, 0.0, 0.6)
    q[::5] = _dense(len(q[::5]), n + 1, counts)
    q[1] = db[5]
    ref = oracle.knn_brute(db, q, k)
    dbt, qt = _t(db), _t(q)
    tree = qd.tree_build(dbt)
    for what, res in (("sequential", qd.knn_bruteforce(dbt, qt, k)),
                      ("blocked", qd.knn_tree(tree, qt, k, order=qd.ORDER_BLOCKED))):
        for got, want in zip(res, (ref.idx.view(np.int32), ref.missed, ref.extra, ref.dist)):
            assert np.array_equal(got.cpu().numpy(), want), what
