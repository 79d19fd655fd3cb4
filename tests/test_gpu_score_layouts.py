"""Object scores for every layout of the rows that the grouping treats apart:
objects in blocks that fill, straddle or fall short of a 1,024-row run, two
objects per 64 rows, objects in turn, and rows of no object between them; with
one to 129 and 257 descriptors (a half and a whole tile, and one past it)."""
import numpy as np
import pytest

import oracle
import synth

pytestmark = pytest.mark.gpu


def _layout(name):
    if name == "whole runs":
        return np.repeat(np.arange(5), 1024)
    if name == "straddling":
        return np.repeat(np.arange(7), [1000, 1100, 3, 64, 1021, 1, 900])
    if name == "two per 64":
        return np.repeat(np.arange(200) % 9, 32)
    if name == "in turn":
        return np.arange(4099) % 300
    if name == "none between":
        o = np.repeat(np.arange(6), 700)
        o[::3] = 60_000
        return o
    o = np.repeat(np.arange(4), 1500)
    o[1024:2048] = 65_535  # a whole run of no object
    return o


@pytest.mark.parametrize("nq", [1, 128, 129, 257])
@pytest.mark.parametrize("name", ["whole runs", "straddling", "two per 64", "in turn", "none between", "run of none"])
@pytest.mark.parametrize("few", [True, False], ids=["few objects", "9000 objects"])
def test_layouts(name, nq, few):
    import torch
    import paper_2107_03368_amd as qd
    obj = _layout(name).astype(np.uint16)
    n_obj = int(obj[obj < 1000].max()) + 1 if few else 9000  # up to 8,192 objects are grouped in LDS
    db = synth.gen_db(len(obj), 3300 + nq)
    q, _ = synth.gen_queries(db, nq, 3301, 0.1, 0.6)
    off = np.array([0, nq // 3, nq // 3, nq], np.uint64)
    ref = oracle.object_scores(db, obj, n_obj, q, off)
    t = lambda a, dt: torch.from_numpy(a.view(dt)).to("cuda:0")
    got = qd.object_scores(t(db, np.int64), t(obj, np.int16), n_obj, t(q, np.int64), t(off, np.int64)).cpu().numpy()
    assert np.array_equal(got, ref)
