"""The projection's two kernels (contraction split over the waves; one chunk
per wave) at the edges of their token tiles and chunks: lengths around 16, 64
and 256 tokens, empty examples, NaN padding, widths of one K-group, one chunk
per example (written straight to the output) and many.  At these sizes the
pooled calls take the split kernel and the per-token calls whichever their own
rule names; the pooled general kernel on ragged rows is compared with the split
one in test_gpu_project_routes.py.  The multi-chunk calls run twice: with the
queried workspace and with the least that the call accepts, which holds the
partials of fewer chunks, so that they run in several rounds.  Bars: 1e-5 relative L2
per row for fp32 (sums of at most 2048 fp32 terms and products: 2^-24 sqrt(2048)
= 2.7e-6), 1e-4 for bf16 (inputs exact, the same sums); a token's block has the
same bars."""
import ctypes
import re

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


def _expect(hm, T, lengths, offs):
    blocks = []
    for a, g, R, S in hm:
        pick = lambda x: np.stack([np.concatenate([x[o:o + n], np.zeros((T - n, x.shape[1]), x.dtype)])
                                   for o, n in zip(offs, lengths)])
        blocks.append(O.project(pick(a), pick(g), R, S, length=lengths))
    return O.project_concat(blocks)


def _least_ws(mods, k, n, T, out, ro, ln, dt):
    L, cm = P.lib(), P._cmods(mods)
    args = (cm, len(mods), dt, k, n, T, ro.data_ptr(), ln.data_ptr(), out.data_ptr(), out.stride(0))
    assert L.attr_project(*args, None, 0, None) == 4
    need = int(re.search(rb"needs (\d+)", L.attr_last_error()).group(1))
    ws = torch.empty(need, dtype=torch.uint8, device="cuda")
    assert L.attr_project(*args, ctypes.c_void_p(ws.data_ptr()), need, P._stream(None)) == 0
    torch.cuda.synchronize()


@pytest.mark.parametrize("dtype", ["bf16", "f32"])
@pytest.mark.parametrize("k", [16, 32, 64])
@pytest.mark.parametrize("T,lengths", [(16, [16, 1, 0]), (64, [64, 15, 17, 0]), (65, [65, 64, 63, 1]),
                                       (300, [300, 0, 257, 256, 255, 48, 129]), (530, [529])])
def test_kernels_at_tile_and_chunk_edges(dtype, k, T, lengths):
    say(f"case: projection {dtype} k={k} T={T} lengths={lengths}")
    rng = np.random.default_rng([k, T])
    shapes = [(64, 64, "x"), (64, 192, "x"), (320, 128, "y"), (64, 64, "z")]
    n, D = len(lengths), len(shapes) * k * k
    lengths = np.array(lengths)
    offs = np.concatenate([[0], np.cumsum(lengths)[:-1]]).astype(np.int64)
    hm, mods = _mods(rng, int(lengths.sum()) + 1, shapes, k, dtype)
    ro, ln = torch.from_numpy(offs).cuda(), torch.from_numpy(lengths.astype(np.int32)).cuda()
    ref = _expect(hm, T, lengths, offs)
    bar = 1e-5 if dtype == "f32" else 1e-4
    out = torch.full((n, D), 7.0, device="cuda")
    P.attr_project(mods, k, n, T, out, row_offset=ro, length=ln)
    got = host(out)
    assert (got[lengths == 0] == 0).all()
    some = lengths > 0
    assert row_rel_l2(got[some], ref[some]).max() <= bar
    if T > 64:
        out.fill_(7.0)
        _least_ws(mods, k, n, T, out, ro, ln, P._dtype(mods[0].a))
        got = host(out)
        assert (got[lengths == 0] == 0).all()
        assert row_rel_l2(got[some], ref[some]).max() <= bar
    # per-token blocks: their sum over an example's tokens is its row
    rows = int(lengths.sum())
    tok = torch.full((rows, D), 7.0, device="cuda")
    P.attr_project_tokens(mods, k, n, T, tok, row_offset=ro, length=ln, ws=P.Workspace("cuda"))
    t = host(tok).astype(np.float64)
    sums = np.stack([t[o:o + m].sum(0) for o, m in zip(offs, lengths)])
    assert row_rel_l2(sums[some], ref[some]).max() <= bar


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
