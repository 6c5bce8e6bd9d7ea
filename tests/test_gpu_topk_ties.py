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


@pytest.mark.parametrize("nq,n,D", PLANS + [(1, 32000, 1024), (1, 600, 64), (3, 300000, 256),
                                             (130, 16385, 64), (130, 65537, 64)])
@pytest.mark.parametrize("dt", [torch.float16, torch.float32])
@pytest.mark.parametrize("k", [1, 10, 100, 128])
@pytest.mark.parametrize("merge", [False, True])
def test_mass_ties(nq, n, D, dt, k, merge):
    """An all-zero query (every score 0), one whose scores take three values, and an
    ordinary one, on integers (exact scores): the list is the stable sort's."""
    if n > 200000 and dt == torch.float32 and k != 100:
        pytest.skip("one k of the large fp32 store")
    say(f"case: ties nq={nq} n={n} D={D} {dt} k={k} merge={merge}")
    g = torch.Generator(device="cuda").manual_seed(n + k)
    G = torch.randint(-2, 3, (n, D), generator=g, device="cuda").to(dt)
    G[:, 0] = torch.randint(0, 3, (n,), generator=g, device="cuda").to(dt)
    Q = torch.zeros((nq, D), dtype=dt, device="cuda")
    if nq > 1:
        Q[1, 0] = 1
    if nq > 2:
        Q[2:] = torch.randint(-2, 3, (nq - 2, D), generator=g, device="cuda").to(dt)
    prev = ([2.0, 2.0, 0.0, -1.0][:k], [4, 900, 17, 2][:k]) if merge else None
    ts, ti = _topk(Q, G, k, prev)
    S = Q.float() @ G.float().T
    idx = torch.arange(1000, 1000 + n, device="cuda").expand(nq, n)
    if merge:
        s, i = (torch.tensor(x, device="cuda").expand(nq, len(x)) for x in prev)
        S, idx = torch.cat([s.float(), S], 1), torch.cat([i, idx], 1)
        order = torch.argsort(idx, dim=1, stable=True)
        S, idx = S.gather(1, order), idx.gather(1, order)
    order = torch.sort(S, dim=1, descending=True, stable=True).indices[:, :k]
    assert torch.equal(ts, S.gather(1, order)) and torch.equal(ti, idx.gather(1, order))


@pytest.mark.parametrize("n", [1, 7, 40, 256, 257])
@pytest.mark.parametrize("dt", [torch.float16, torch.float32])
@pytest.mark.parametrize("k", [8, 9, 100, 128])
@pytest.mark.parametrize("merge", [False, True])
def test_fewer_rows_than_k(n, dt, k, merge):
    """Stores of few rows, some of them NaN or infinite, on both sides of the small
    store's rule: every row but NaN and -inf, then empty entries."""
    say(f"case: few rows n={n} {dt} k={k} merge={merge}")
    g = torch.Generator(device="cuda").manual_seed(n + k)
    G = torch.randint(-2, 3, (n, 192), generator=g, device="cuda").to(dt)
    Q = torch.randint(-2, 3, (5, 192), generator=g, device="cuda").to(dt)
    Q[:, 0] = 1
    G[n // 2, 0], G[n // 3, 0], G[0, 0] = float("nan"), -float("inf"), float("inf")
    prev = ([3.0, 0.0, -0.0][:k], [5, 3000, 7000][:k]) if merge else None
    ts, ti = _topk(Q, G, k, prev)
    # (-inf for what is never selected; NaN products of inf and 0 cannot arise in column 0)
    S = (Q.float().unsqueeze(1) * G.float()).sum(2)
    idx = torch.arange(1000, 1000 + n, device="cuda").expand(5, n)
    if merge:
        s, i = (torch.tensor(x, device="cuda").expand(5, len(x)) for x in prev)
        S, idx = torch.cat([s.float(), S], 1), torch.cat([i, idx], 1)
    for q in range(5):
        live = [(-s, i) for s, i in zip(S[q].tolist(), idx[q].tolist()) if s > -float("inf")]
        want = sorted((s + 0.0, i) for s, i in live)[:k]
        want += [(float("inf"), -1)] * (k - len(want))
        assert ti[q].tolist() == [i for _, i in want]
        assert ts[q].tolist() == [-s for s, _ in want]
