"""Node splits of the tree build at the edges of their kernels: nodes held in
registers (up to 128 rows), read twice by one block (up to 2,048) and shared by
several blocks; rows whose least popular bits reach half the node at the first
try and rows where they do not.  Trees equal the oracle's, as integers."""
import numpy as np
import pytest

import oracle
import synth

pytestmark = pytest.mark.gpu


def _rows(kind, n):
    if kind == "generated":
        return synth.gen_db(n, 4000 + n)
    rng = np.random.default_rng(n)
    bits = np.zeros((n, 4096), np.uint8)
    bits[:, :200] = rng.random((n, 200)) < 0.9
    dense = rng.choice(n, max(1, n // 40), replace=False)
    bits[dense] = rng.random((len(dense), 4096)) < 0.75  # a few rows hold every rare bit
    if kind == "outliers and empty rows":  # fewer than half the rows have a bit at all
        empty = rng.choice(n, (6 * n) // 10, replace=False)
        bits[empty] = 0
    return np.packbits(bits, axis=1, bitorder="little").view(np.uint64)


@pytest.mark.parametrize("kind", ["generated", "outliers", "outliers and empty rows"])
@pytest.mark.parametrize("n", [33, 64, 65, 127, 128, 129, 257, 1000, 2047, 2048, 2049, 3073, 9000])
def test_split_edges(n, kind):
    import paper_2107_03368_amd as qd
    import torch
    db = _rows(kind, n)
    ot = oracle.tree_build(db)
    gt = qd.tree_build(torch.from_numpy(db.view(np.int64)).to("cuda:0")).export()
    for key, ref in (("child", ot.child), ("begin", ot.begin), ("count", ot.count), ("perm", ot.perm),
                     ("or_img", ot.or_img)):
        assert np.array_equal(gt[key].astype(ref.dtype), ref), key
