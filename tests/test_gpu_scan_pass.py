"""The matrix pass of the sequential search at its edges: query counts around
the 64-query tiles and 256-query groups, rows around the 64-row tiles, sampled
bounds that mislead (rows in order of distance), hundreds to thousands of
candidates tied at the k-th key, overflowing buffers, and passes in several
parts; against the oracle, or the vector row scan where that is too slow."""
import numpy as np
import pytest

import oracle
import synth

pytestmark = pytest.mark.gpu


def _t(a):
    import torch
    return torch.from_numpy(np.ascontiguousarray(a).view(np.int64)).to("cuda:0")


def _check(db, q, k):
    import paper_2107_03368_amd as qd
    ref = oracle.knn_brute(db, q, k)
    for got, want in zip(qd.knn_bruteforce(_t(db), _t(q), k), (ref.idx.view(np.int32), ref.missed, ref.extra, ref.dist)):
        assert np.array_equal(got.cpu().numpy(), want)


@pytest.mark.parametrize("nq", [9, 17, 63, 64, 65, 129, 192, 255, 256, 257, 300, 321, 513])
def test_query_counts(nq):
    db = synth.gen_db(8_255, 800)
    q, _ = synth.gen_queries(db, nq, 801 + nq, 0.0, 0.6)
    q[nq // 2] = 0
    q[nq // 3] = ~np.uint64(0)
    _check(db, q, 10)


@pytest.mark.parametrize("n", [8_192, 8_193, 8_255, 8_256, 16_383, 16_385, 40_001])
@pytest.mark.parametrize("k", [5, 31])
def test_row_counts(n, k):
    db = synth.gen_db(n, 810)
    q, _ = synth.gen_queries(db, 20, 811, 0.1, 0.6)
    _check(db, q, k)


def test_few_neighbours_from_many_pairs():
    db = synth.gen_db(131_073, 815)
    q, _ = synth.gen_queries(db, 257, 816, 0.1, 0.6)
    _check(db, q, 1)
    _check(db, q, 3)


@pytest.mark.parametrize("tied", [200, 300, 1_500, 8_000, 9_000])
def test_ties_at_the_kth_key(tied):
    # the query's nearest rows: 4 closer ones, then `tied` equal rows of which 6 belong to the top 10
    db = synth.gen_db(16_000, 820)
    rng = np.random.default_rng(821)
    at = np.sort(rng.choice(16_000, tied + 4, replace=False))
    base = db[0].copy()
    db[at] = base
    db[at[::-1][:4]] = base
    q = np.tile(base, (20, 1))
    q[:, 0] ^= np.arange(20, dtype=np.uint64)
    for i, r in enumerate(rng.choice(at, 4, replace=False)):
        db[r, 0] = q[i + 1, 0]
    _check(db, q, 10)


@pytest.mark.parametrize("order", ["near rows last", "near rows first"])
def test_rows_in_order_of_distance(order):
    db = synth.gen_db(60_000, 830)
    q, _ = synth.gen_queries(db, 40, 831, 0.1, 0.4)
    p = np.argsort(np.bitwise_count(db & q[0]).sum(1), kind="stable")
    db = db[p if order == "near rows last" else p[::-1]]
    _check(db, q, 20)


@pytest.mark.parametrize("n,nq,k", [(300_001, 4_097, 10), (1_000_001, 600, 1), (600_000, 2_000, 50)])
def test_passes_in_parts(n, nq, k):
    import torch
    import paper_2107_03368_amd as qd
    db = synth.gen_db(n, 840)
    q, _ = synth.gen_queries(db, nq, 841, 0.1, 0.6)
    dbt, qt = _t(db), _t(q)
    res = qd.knn_bruteforce(dbt, qt, k)
    ref = qd.knn_bruteforce(dbt, qt, k, query_tile=16)
    assert all(torch.equal(a, b) for a, b in zip(res, ref))
    some = np.arange(0, nq, max(1, nq // 4))
    o = oracle.knn_brute(db, q[some], k)
    assert np.array_equal(res[0].cpu().numpy()[some].view(np.uint32), o.idx)
