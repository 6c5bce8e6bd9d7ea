"""The selection kernels at the sizes where their register layouts change: 1024,
4096 and 16384 rows per query (one, four and sixteen rows per thread), 16 and 32
queries per block, lists shorter and longer than the store, a previous list,
NaN rows, and merges of few long and many short lists.  Scores are dot products of
unit rows in fp32 accumulation, compared with fp64 to 1e-3 as everywhere; the
order rule is the oracle's."""
import re

import numpy as np
import pytest
import torch

import oracle as O
import paper_2606_11660_amd as P
import synth
from tests._util import check_topk, dev, host, say

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("nq,ng,k,dt", [
    (1, 257, 1, np.float16), (16, 1023, 128, np.float16), (17, 1024, 100, np.float32), (5, 1025, 10, np.float16),
    (33, 4096, 100, np.float16), (2, 4097, 128, np.float32), (32, 16384, 5, np.float16), (3, 16385, 100, np.float16),
    (1, 32000, 128, np.float16)])
@pytest.mark.parametrize("merge", [False, True])
def test_split_selection_edges(nq, ng, k, dt, merge):
    say(f"case: split selection nq={nq} ng={ng} k={k} {dt.__name__} merge={merge}")
    D = 1024
    Q, G = synth.unit_rows(nq, D, seed=nq).astype(dt), synth.unit_rows(ng, D, seed=ng).astype(dt)
    G[ng // 2, 3] = np.nan
    ref = O.scores(Q.astype(np.float32), G.astype(np.float32))
    cut = ng // 3 if merge else 0
    ts = torch.empty((nq, k), dtype=torch.float32, device="cuda")
    ti = torch.empty((nq, k), dtype=torch.int64, device="cuda")
    Qd, Gd = dev(Q), dev(G)
    if merge:
        P.attr_score_topk(Qd, Gd[:cut], k, ts, ti)
    P.attr_score_topk(Qd, Gd[cut:], k, ts, ti, index_base=cut, merge=merge)
    check_topk(host(ts), host(ti), np.where(np.isnan(ref), -np.inf, ref), k)


@pytest.mark.parametrize("nq,ng,D,k,dt", [(8, 256, 256, 5, np.float32), (1, 100, 64, 10, np.float16),
                                          (70, 2000, 512, 100, np.float16), (20, 9000, 256, 128, np.float16),
                                          (100, 3001, 448, 128, np.float32), (16, 5000, 960, 1, np.float16)])
@pytest.mark.parametrize("merge", [False, True])
def test_narrow_rows_with_the_queried_and_the_least_workspace(nq, ng, D, k, dt, merge):
    """Few, narrow rows take the split plan's kernels; a workspace that holds only
    the streaming plan's lists takes that plan, with the same answer."""
    say(f"case: narrow rows nq={nq} ng={ng} D={D} k={k} {dt.__name__} merge={merge}")
    Q, G = synth.unit_rows(nq, D, seed=3).astype(dt), synth.unit_rows(ng, D, seed=4).astype(dt)
    G[ng - 1] = G[5]
    ref = O.scores(Q.astype(np.float32), G.astype(np.float32))
    cut = ng // 2 if merge else 0
    Qd, Gd = dev(Q), dev(G)
    L, code = P.lib(), P.ATTR_F16 if dt == np.float16 else P.ATTR_F32
    for least in (False, True):
        ts = torch.empty((nq, k), dtype=torch.float32, device="cuda")
        ti = torch.empty((nq, k), dtype=torch.int64, device="cuda")
        for lo, hi, m in ((0, cut, 0), (cut, ng, int(merge))):
            if lo == hi:
                continue
            if not least:
                P.attr_score_topk(Qd, Gd[lo:hi], k, ts, ti, index_base=lo, merge=bool(m))
                continue
            args = (Qd.data_ptr(), nq, D, Gd[lo:].data_ptr(), hi - lo, D, code, D, k, lo, m, ts.data_ptr(),
                    ti.data_ptr())
            assert L.attr_score_topk(*args, None, 0, None) == 4
            need = int(re.search(rb"needs (\d+)", L.attr_last_error()).group(1))
            assert need <= P.attr_score_topk_workspace_size(nq, hi - lo, D, k)
            ws = torch.empty(need, dtype=torch.uint8, device="cuda")
            assert L.attr_score_topk(*args, ws.data_ptr(), need, P._stream(None)) == 0
            torch.cuda.synchronize()
        check_topk(host(ts), host(ti), ref, k)


@pytest.mark.parametrize("nq,ng,D,k,dt", [(3, 40000, 64, 128, np.float16),      # 313 lists and the previous one
                                          (130, 9000, 64, 100, np.float16),     # one chunk's list and the previous one
                                          (70, 33000, 64, 25, np.float32)])
def test_merge_of_lists_and_a_previous_list(nq, ng, D, k, dt):
    say(f"case: merge nq={nq} ng={ng} k={k}")
    Q, G = synth.unit_rows(nq, D, seed=1).astype(dt), synth.unit_rows(ng, D, seed=2).astype(dt)
    G[7] = G[ng - 1]  # a tie across the lists
    prev_s = np.full((nq, k), -np.inf, np.float32)
    prev_i = np.full((nq, k), -1, np.int64)
    prev_s[:, 0], prev_i[:, 0] = 0.5, 3          # a valid head
    prev_s[0, 1], prev_i[0, 1] = -np.inf, 4      # a valid index under -inf stays last
    ts, ti = dev(prev_s), dev(prev_i)
    P.attr_score_topk(dev(Q), dev(G), k, ts, ti, index_base=1000, merge=True)
    ref = O.scores(Q.astype(np.float32), G.astype(np.float32))
    ref = np.concatenate([np.full((nq, 1000), -np.inf), ref], 1)
    ref[:, 3] = 0.5
    check_topk(host(ts), host(ti), ref, k)
