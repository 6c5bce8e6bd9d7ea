"""Ties in the top-k: equal scores are ordered by index, whatever kernel selects them
(a store of up to 256 rows, the split selection, the merge of the streaming and of the
GEMM plan's lists), and -0 equals +0."""
import numpy as np
import pytest
import torch

import paper_2606_11660_amd as P
from tests._util import say

pytestmark = pytest.mark.gpu

PLANS = [(3, 200, 512), (3, 4000, 512), (3, 20000, 1024), (5, 40000, 64), (130, 9000, 64), (2, 270000, 64)]


def _topk(Q, G, k, prev=None):
    nq = Q.shape[0]
    ts = torch.full((nq, k), -float("inf"), device="cuda")
    ti = torch.full((nq, k), -1, dtype=torch.int64, device="cuda")
    if prev:
        s, i = prev
        ts[:, :len(s)] = torch.tensor(s, device="cuda")
        ti[:, :len(i)] = torch.tensor(i, device="cuda")
    P.attr_score_topk(Q, G, k, ts, ti, index_base=1000, merge=prev is not None)
    return ts, ti


@pytest.mark.parametrize("nq,n,D", PLANS)
@pytest.mark.parametrize("dt", [torch.float16, torch.float32])
@pytest.mark.parametrize("k", [1, 5])
def test_zeros_of_either_sign_are_equal(nq, n, D, dt, k):
    say(f"case: signed zeros nq={nq} n={n} D={D} {dt} k={k}")
    Q = torch.zeros((nq, D), dtype=dt, device="cuda")
    G = torch.ones((n, D), dtype=dt, device="cuda")
    ts, ti = _topk(Q, G, k, prev=([-0.0, -0.0][:k], [3, 7][:k]))
    want = ([3, 7] + list(range(1000, 1000 + k)))[:k]
    assert (ti == torch.tensor(want, device="cuda")).all() and (ts == 0).all()
