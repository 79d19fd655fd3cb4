"""The merge of a scan's lists when every list's first row ties: no list but those
of the k nearest is left to order, so it costs about what it costs otherwise."""
import numpy as np
import pytest

import synth

pytestmark = pytest.mark.gpu


# 1,560 and 4,096 lists whose heads were all sorted: 7 to 9 times the time.
@pytest.mark.parametrize("n,nq,k", [(400_000, 1, 1), (400_000, 2, 10), (100_000, 1, 10)])
def test_tied_heads_cost_no_more(n, nq, k):
    import torch
    import paper_2107_03368_amd as qd

    def merge_ms(db, q):
        qd.knn_bruteforce(db, q, k)
        torch.cuda.synchronize()
        qd.profile_enable(True)
        try:
            for _ in range(20):
                qd.knn_bruteforce(db, q, k)
            torch.cuda.synchronize()
            ms, launches = qd.profile_read("topk_merge")
        finally:
            qd.profile_enable(False)
        return ms / launches

    db = torch.from_numpy(synth.gen_db(n, 980).view(np.int64)).to("cuda:0")
    q = torch.from_numpy(synth.gen_queries(synth.gen_db(100, 980), nq, 981, 0.1, 0.5)[0].view(np.int64)).to("cuda:0")
    plain = merge_ms(db, q)
    db[:] = db[3].clone()
    assert merge_ms(db, q) < 3 * plain
    assert qd.knn_bruteforce(db, q, k)[0].tolist() == [list(range(k))] * nq
