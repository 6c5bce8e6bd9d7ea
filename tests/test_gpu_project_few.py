"""Per-token blocks in a workspace of exactly the queried size."""
import numpy as np
import pytest
import torch

import oracle as O
import paper_2606_11660_amd as P
import synth
from tests._util import dev, host, row_rel_l2, say

pytestmark = pytest.mark.gpu


def _mods(rng, rows, shapes, k, dtype):
    enc = synth.to_bf16_bits if dtype == "bf16" else (lambda x: x.astype(np.float32))
    hm, dm, shared = [], [], {}
    for m, (d_in, d_out, tag) in enumerate(shapes):
        if tag not in shared:
            a = enc(rng.standard_normal((rows, d_in)))
            a[-1] = enc(np.full((1, d_in), np.nan))[0]
            shared[tag] = (a, dev(a))
        g = enc(rng.standard_normal((rows, d_out)) * 1e-2)
        g[-1] = enc(np.full((1, d_out), np.nan))[0]
        R, S = enc(rng.standard_normal((d_out, k)) / k ** 0.5), enc(rng.standard_normal((d_in, k)) / k ** 0.5)
        hm.append((shared[tag][0], g, R, S))
        dm.append(P.Module(shared[tag][1], dev(g), dev(R), dev(S), out_col=m * k * k))
    return hm, dm


def test_tokens_fit_the_queried_workspace():
    # 42 modules in groups of up to three: the ungrouped per-token call's group
    # table is larger than the grouped one's that the query lays out
    say("case: per-token call in a workspace of the queried size")
    rng = np.random.default_rng(5)
    shapes = [(64, 64, "x%d" % (j // 3)) for j in range(42)]
    hm, mods = _mods(rng, 9, shapes, 16, "bf16")
    out = torch.zeros((8, 42 * 256), device="cuda")
    P.attr_project_tokens(mods, 16, 1, 8, out, ws=P.Workspace("cuda"))
    ref = np.concatenate([O.project(a[None, :8], g[None, :8], R, S).reshape(1, -1) for a, g, R, S in hm], 1)
    assert row_rel_l2(host(out).astype(np.float64).sum(0, keepdims=True), ref).max() <= 1e-4
