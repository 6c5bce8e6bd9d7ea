"""The projection's bits do not depend on the scratch it is given: the queried
workspace, the least that the call accepts (the partials of the few-item kernel
then come in rounds of chunks) and the static array of the allocation-free call
give the same rows.  Sizes: one round and several, rounds that end inside an
example, one 64-token chunk per round, chunks of 16 tokens, and partials past the
static array."""
import ctypes
import re

import pytest
import torch

import paper_2606_11660_amd as P
from tests._util import say

pytestmark = pytest.mark.gpu


def _call(dt, k, n, T, shapes, ragged, seed=0):
    g = torch.Generator(device="cuda").manual_seed(seed + k + T)
    rand = lambda *s: torch.randn(s, generator=g, device="cuda").to(dt)
    mods = [P.Module(rand(n * T, a), rand(n * T, b), rand(b, k), rand(a, k), j * k * k)
            for j, (a, b) in enumerate(shapes)]
    ln = None
    if ragged:
        ln = torch.randint(0, T + 1, (n,), generator=g, device="cuda", dtype=torch.int32)
        ln[0], ln[-1] = T, 0
    return mods, ln


def _least(mods, k, n, T, out, ln):
    L, cm, dt = P.lib(), P._cmods(mods), P._dtype(mods[0].a)
    args = (cm, len(mods), dt, k, n, T, None, P._ptr(ln), out.data_ptr(), out.stride(0))
    assert L.attr_project(*args, None, 0, None) == 4
    need = int(re.search(rb"needs (\d+)", L.attr_last_error()).group(1))
    query = L.attr_project_workspace_size(cm, len(mods), dt, n, T, k)
    ws = torch.empty(need, dtype=torch.uint8, device="cuda")
    assert L.attr_project(*args, ctypes.c_void_p(ws.data_ptr()), need, P._stream(None)) == 0
    torch.cuda.synchronize()
    return need, query


@pytest.mark.parametrize("dt,k,n,T,shapes,ragged", [
    (torch.bfloat16, 16, 1, 700, [(64, 128)] * 3, False),       # 3 chunks' room, 11 chunks
    (torch.bfloat16, 16, 5, 300, [(64, 64), (128, 64)], True),
    (torch.bfloat16, 32, 2, 200, [(64, 128)] * 2, True),        # one chunk per round
    (torch.bfloat16, 64, 3, 1100, [(64, 64)], True),
    (torch.bfloat16, 16, 1, 149, [(2048, 2048)], False),        # 16-token chunks
    (torch.float32, 16, 2, 530, [(96, 64)], True),
    (torch.float32, 32, 4, 257, [(64, 96)] * 2, False),
    (torch.float32, 64, 1, 6400, [(64, 64)] * 48, False),       # 79 MB of partials
])
def test_bits_do_not_depend_on_the_scratch(dt, k, n, T, shapes, ragged):
    say(f"case: projection scratch {dt} k={k} n={n} T={T} modules={len(shapes)} ragged={ragged}")
    mods, ln = _call(dt, k, n, T, shapes, ragged)
    out = [torch.full((n, len(shapes) * k * k), 7.0, device="cuda") for _ in range(3)]
    P.attr_project(mods, k, n, T, out[0], length=ln, ws=P.Workspace("cuda"))
    need, query = _least(mods, k, n, T, out[1], ln)
    assert need < query  # the least workspace holds fewer partials
    P.attr_project_noalloc(mods, k, n, T, out[2], length=ln)
    assert torch.equal(out[0], out[1]) and torch.equal(out[0], out[2])
    if ln is not None:
        assert (out[0][ln == 0] == 0).all()
