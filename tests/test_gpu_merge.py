"""The merge of a scan's lists where its selection can go wrong: more lists
than threads, heads that all tie in K (every list qualifies by K and the row
index decides), fewer rows than k, and 1 .. 4,096 row slices, against the
oracle."""
import numpy as np
import pytest

import oracle
import synth

pytestmark = pytest.mark.gpu


def _t(a):
    import torch
    return torch.from_numpy(np.ascontiguousarray(a).view(np.int64)).to("cuda:0")


def _check(db, q, k, **kw):
    import paper_2107_03368_amd as qd
    ref = oracle.knn_brute(db, q, k)
    res = qd.knn_bruteforce(_t(db), _t(q), k, **kw)
    for got, want in zip(res, (ref.idx.view(np.int32), ref.missed, ref.extra, ref.dist)):
        assert np.array_equal(got.cpu().numpy(), want)


@pytest.mark.parametrize("k", [1, 10, 64])
@pytest.mark.parametrize("n", [1, 15, 17, 64, 4_095, 4_097, 66_000, 200_003])
def test_row_counts(n, k):
    db = synth.gen_db(n, 700)
    q, _ = synth.gen_queries(db, 3, 701, 0.1, 0.5)
    _check(db, q[:1], k)
    _check(db, q, k)


@pytest.mark.parametrize("k", [1, 10, 64])
@pytest.mark.parametrize("rows", ["all equal", "two kinds", "sorted near", "empty and full"])
def test_ties_between_lists(rows, k):
    n = 70_000
    db = synth.gen_db(n, 710)
    q, _ = synth.gen_queries(db, 2, 711, 0.1, 0.5)
    if rows == "all equal":
        db[:] = db[0]
    elif rows == "two kinds":
        db[:] = db[0]
        db[3::17] = q[0]
    elif rows == "sorted near":  # all of the nearest rows in one slice
        db[1_000:1_200] = q[0]
        db[1_100, 0] ^= np.uint64(1)
    else:
        db[::2] = 0
        db[1::2] = ~np.uint64(0)
        q[1] = 0
    _check(db, q, k)
    _check(db, q, k, query_tile=16, row_parts=273)
