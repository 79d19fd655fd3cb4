"""Rows that tie at a query's k-th key (repeated or blank descriptors, blank
queries) in the matrix pass of the sequential search: the answers, against the
vector row scan and the oracle, and the time, against the same shape without
ties."""
import statistics

import numpy as np
import pytest

import oracle
import synth

pytestmark = pytest.mark.gpu

K = 10


def _t(a):
    import torch
    return torch.from_numpy(np.ascontiguousarray(a).view(np.int64)).to("cuda:0")


def _corner(nq):
    """Queries of bits that no generated row has: every row misses all of them, and a blank row adds none."""
    q = np.zeros((nq, 64), np.uint64)
    q[:, 0] = 7
    q[:, 1] = 3
    q[:, 63] = 7
    return q


def _ms(db, q, k):
    import torch
    import paper_2107_03368_amd as qd
    qd.knn_bruteforce(db, q, k)
    times = []
    for _ in range(7):
        a, b = (torch.cuda.Event(enable_timing=True) for _ in range(2))
        a.record()
        qd.knn_bruteforce(db, q, k)
        b.record()
        torch.cuda.synchronize()
        times.append(a.elapsed_time(b))
    return statistics.median(times)


# The pass in parts (4,097 queries): its first part ends after 65,536 rows.
@pytest.mark.parametrize("first", [20_000, 60_000, 250_000])
def test_tied_rows_in_parts(first):
    import torch
    import paper_2107_03368_amd as qd
    n, nq, tied = 300_001, 4_097, 9_000
    db = synth.gen_db(n, 850)
    q, _ = synth.gen_queries(db, nq, 851, 0.1, 0.6)
    base = db[7].copy()
    db[first:first + tied] = base
    some = np.array([0, 1, 255, 256, 777, 2_048, 4_096])  # equal to the row, blank, and far from every row
    q[some[0::3]] = base
    q[some[1::3]] = 0
    q[some[2::3]] = _corner(1)
    db[::100] = 0
    dbt, qt = _t(db), _t(q)
    res = qd.knn_bruteforce(dbt, qt, K)
    ref = qd.knn_bruteforce(dbt, qt, K, query_tile=16)
    assert all(torch.equal(a, b) for a, b in zip(res, ref))
    o = oracle.knn_brute(db, q[some], K)
    assert np.array_equal(res[0].cpu().numpy()[some].view(np.uint32), o.idx)


# Listing every tied row took some 17 times the time of the same shape without ties.
@pytest.mark.parametrize("nq,k", [(64, 10), (64, 1), (1_024, 10)])
def test_blank_rows_cost_no_more(nq, k):
    n = 2_000_000
    db = synth.gen_db(n, 860)
    dbt, qt = _t(db), _t(_corner(nq))
    plain = _ms(dbt, qt, k)
    dbt[np.random.default_rng(861).choice(n, n // 50, replace=False)] = 0
    assert _ms(dbt, qt, k) < 3 * plain


# Whole tiles sampled: these took 3 to 17 times the time without.
@pytest.mark.parametrize("nq,k", [(64, 10), (64, 1), (1_024, 10), (1_024, 1)])
@pytest.mark.parametrize("rows", ["equal", "a run of blanks", "by distance"])
def test_runs_of_similar_rows_cost_no_more(rows, nq, k):
    import torch
    import paper_2107_03368_amd as qd
    n = 1_000_000
    db = synth.gen_db(n, 870)
    q, _ = synth.gen_queries(db, nq, 871, 0.1, 0.4)
    dbt, qt = _t(db), _t(q)
    plain = _ms(dbt, qt, k)
    if rows == "equal":
        dbt[:] = dbt[5].clone()
    elif rows == "a run of blanks":
        dbt[n // 2:n // 2 + n // 20] = 0
        qt = _t(_corner(nq))
    else:
        p = np.argsort(-np.bitwise_count(db & q[0]).sum(1, dtype=np.int64), kind="stable")
        dbt = dbt[torch.from_numpy(p).to(dbt.device)].contiguous()
        q[:] = q[0]
        q[:, 40] ^= np.arange(nq, dtype=np.uint64) % np.uint64(64)
        qt = _t(q)
    assert _ms(dbt, qt, k) < 2 * plain
    res, ref = qd.knn_bruteforce(dbt, qt, k), qd.knn_bruteforce(dbt, qt, k, query_tile=16)
    assert all(torch.equal(a, b) for a, b in zip(res, ref))


@pytest.mark.parametrize("period", [8, 50, 64, 512, 3_264])
def test_periodic_rows(period):
    # near rows at every period-th place
    import paper_2107_03368_amd as qd
    db = synth.gen_db(200_000, 880)
    q, _ = synth.gen_queries(db, 33, 881, 0.1, 0.4)
    noise = np.random.default_rng(882).integers(0, 2**64, (len(db[3::period]), 64), dtype=np.uint64)
    for i in range(1, 5):
        noise &= np.roll(noise, i, 1)
    db[3::period] = q[0] | noise
    q[:] = q[0]
    q[:, 5] ^= np.arange(33, dtype=np.uint64)
    o = oracle.knn_brute(db, q, K)
    res = qd.knn_bruteforce(_t(db), _t(q), K)
    assert np.array_equal(res[0].cpu().numpy().view(np.uint32), o.idx)
    assert np.array_equal(res[3].cpu().numpy(), o.dist)


def _sampled(n, k):
    """The rows that a pass in one part samples."""
    tiles = min((max(n // 512 * k, 128 * k, min(n // 512 * 16, 32_768)) + 63) // 64, (n + 63) // 64, 4096)
    step = (n << 32) // (64 * tiles)
    i = np.arange(64 * tiles + 1, dtype=np.uint64)
    a = (i * np.uint64(step)) >> np.uint64(32)
    m = np.uint64(0xFFFFFFFF)
    h = (i * np.uint64(2654435761)) & m
    h = ((h ^ (h >> np.uint64(16))) * np.uint64(2654435761)) & m
    return (a[:-1] + ((h[:-1] * (a[1:] - a[:-1])) >> np.uint64(32))).astype(np.int64)


# Rows that the sample misses fill the buffers: the queries are passed over the
# rows again, and once more by one workgroup each where the rows that come first
# in every workgroup's run are farther than the others.
@pytest.mark.parametrize("twice", [False, True])
@pytest.mark.parametrize("n,nq,k", [(300_000, 20, 4), (263_007, 70, 10)])
def test_overflowing_buffers(n, nq, k, twice):
    import torch
    import paper_2107_03368_amd as qd
    rng = np.random.default_rng(890)
    db = synth.gen_db(n, 890)
    base = db[11].copy()
    bits = np.flatnonzero(np.unpackbits(base.view(np.uint8), bitorder="little"))
    far = np.zeros(n, bool)
    far[_sampled(n, k)] = True

    def near(rows, lost):  # copies of the base that lack `lost` or more of its bits
        b = np.tile(np.unpackbits(base.view(np.uint8), bitorder="little"), (len(rows), 1))
        for i in range(lost + 3):
            b[np.arange(len(rows)), rng.choice(bits, len(rows)) if i >= lost else bits[i]] = 0
        db[rows] = np.packbits(b, axis=1, bitorder="little").view(np.uint64)

    if twice:
        cus = torch.cuda.get_device_properties(0).multi_processor_count
        units = (n + 63) // 64 * ((nq + 63) // 64)
        start = np.array([units // cus * b + min(b, units % cus) for b in range(cus + 1)]) // ((nq + 63) // 64)
        tile = np.arange(n) // 64
        late = tile - start[np.searchsorted(start, tile, side="right") - 1] >= 8 // ((nq + 63) // 64)
        near(np.flatnonzero(~far & late), 1)
        near(np.flatnonzero(~far & ~late), 20)
    else:
        near(rng.choice(np.flatnonzero(~far), 20_000, replace=False), 2)
    q = np.tile(base, (nq, 1))
    q[:, 0] ^= np.arange(nq, dtype=np.uint64)
    q[nq // 2] = synth.gen_queries(db[:100], 1, 891, 0.1, 0.3)[0][0]
    dbt, qt = _t(db), _t(q)
    res = qd.knn_bruteforce(dbt, qt, k)
    ref = qd.knn_bruteforce(dbt, qt, k, query_tile=16)
    assert all(torch.equal(a, b) for a, b in zip(res, ref))
    some = np.array([0, 1, nq // 2, nq - 1])
    o = oracle.knn_brute(db, q[some], k)
    assert np.array_equal(res[0].cpu().numpy()[some].view(np.uint32), o.idx)
    assert np.array_equal(res[3].cpu().numpy()[some], o.dist)


@pytest.mark.parametrize("n,views", [(192_000, 3_000), (640_000, 10_000), (131_072, 2_048)])
def test_near_rows_at_one_place_of_every_object(n, views):
    # 64 objects of so many views; the nearest are some neighbouring views of all
    import paper_2107_03368_amd as qd
    import torch
    rng = np.random.default_rng(895)
    db = synth.gen_db(n, 895)
    base = db[5].copy()
    bits = np.flatnonzero(np.unpackbits(base.view(np.uint8), bitorder="little"))
    rows = (np.arange(64)[:, None] * views + views // 3 + np.arange(60)[None]).reshape(-1)
    b = np.tile(np.unpackbits(base.view(np.uint8), bitorder="little"), (len(rows), 1))
    for _ in range(12):
        b[np.arange(len(rows)), rng.choice(bits, len(rows))] = 0
    db[rows] = np.packbits(b, axis=1, bitorder="little").view(np.uint64)
    q = np.tile(base, (40, 1))
    q[:, 0] ^= np.arange(40, dtype=np.uint64)
    dbt, qt = _t(db), _t(q)
    for k in (1, 10, 64):
        res, ref = qd.knn_bruteforce(dbt, qt, k), qd.knn_bruteforce(dbt, qt, k, query_tile=16)
        assert all(torch.equal(x, y) for x, y in zip(res, ref))
