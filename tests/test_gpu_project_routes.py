"""Calls large enough for the general projection kernel, on narrow modules: the
plan depends on the widths' proportions, so layers shaped as a 1B model's, 32 times
narrower, take the kernels that the model's would.  ROUTES names the kernel that
each case takes (checked on the CPU, in test_project_plan_cpu.py): groups of three,
two and one in the general kernel, and both sides of the line between the kernels,
shared input rows against separate copies; TOKEN_ROUTES the same for per-token
calls; WIDE few tokens through wide modules, 16 tokens per workgroup.  References in fp64 on the GPU; bars as
in test_gpu_project_few.py: 1e-5 relative L2 per row for fp32, 1e-4 for bf16."""
import pytest
import torch

import paper_2606_11660_amd as P
from tests._util import say

pytestmark = pytest.mark.gpu

# d_in, d_out and the rows a module reads (same tag in one layer: the same rows)
LAYER = ((64, 64, "x"), (64, 64, "x"), (64, 64, "x"), (64, 64, "o"), (64, 256, "m"), (64, 256, "m"), (256, 64, "d"))

# dtype, k, layers, examples, T, lengths given, kernel
ROUTES = [("bf16", 16, 2, 16, 2048, False, "general"), ("bf16", 16, 2, 20, 2048, True, "general"),
          ("bf16", 16, 3, 100, 300, False, "general"),
          ("bf16", 32, 2, 8, 2048, False, "general"), ("bf16", 32, 2, 12, 2048, True, "general"),
          ("bf16", 64, 2, 5, 2048, False, "general"), ("bf16", 64, 1, 20, 1030, True, "general"),
          ("f32", 16, 2, 16, 2048, False, "general"), ("f32", 16, 2, 20, 2048, True, "general"),
          # next to the line, where a rule with the shared widths would take another
          # kernel than for separate copies
          ("bf16", 16, 2, 8, 2048, False, "general"), ("bf16", 16, 1, 16, 2048, False, "general"),
          ("bf16", 16, 2, 9, 2048, False, "general"), ("bf16", 16, 2, 32, 512, False, "general"),
          ("bf16", 16, 4, 4, 2048, False, "general"), ("bf16", 16, 2, 16, 2048, True, "general"),
          ("bf16", 16, 2, 4, 2048, False, "few 64"), ("bf16", 16, 2, 8, 2048, True, "few 64"),
          ("bf16", 32, 2, 4, 2048, False, "few 64"), ("bf16", 64, 2, 2, 1024, False, "few 64"),
          ("f32", 16, 2, 7, 2048, False, "few 64"), ("f32", 32, 2, 5, 700, True, "few 64"),
          ("f32", 64, 2, 3, 700, False, "few 64")]


TOKEN_ROUTES = [("bf16", 16, 2, 16, 2048, False, "general"), ("bf16", 16, 2, 20, 2048, True, "general"),
                ("bf16", 32, 2, 4, 2048, False, "general"), ("bf16", 32, 2, 7, 1500, True, "general"),
                ("bf16", 64, 1, 5, 1030, False, "general"), ("bf16", 64, 1, 10, 700, True, "general"),
                ("f32", 16, 2, 16, 2048, False, "general"), ("f32", 16, 2, 20, 2048, True, "general"),
                ("bf16", 16, 2, 2, 2048, False, "few 64"), ("bf16", 32, 1, 3, 600, True, "few 64"),
                ("bf16", 64, 1, 3, 300, True, "few 64"), ("f32", 32, 1, 4, 700, True, "few 64")]

# shapes, examples, T, lengths
WIDE = [([(2048, 2048)], 1, 1, None), ([(2048, 2048)], 1, 16, None), ([(4096, 8704)], 1, 17, None),
        ([(4096, 8704), (4096, 4096)], 1, 149, None), ([(2048, 2048)], 1, 16, [15]), ([(2048, 2048)], 2, 1, [0, 1]),
        ([(8192, 6400), (2048, 6400)], 3, 40, [33, 0, 16]), ([(8192, 4608)], 2, 149, [149, 130])]


def make(dt, k, layers, n, T, ragged, shared=True, layer=LAYER, lengths=None):
    dtype = torch.bfloat16 if dt == "bf16" else torch.float32
    g = torch.Generator(device="cuda").manual_seed(k + n + T)
    rand = lambda *s: torch.randn(s, generator=g, device="cuda")
    ln = None
    if lengths:
        ln = torch.tensor(lengths, device="cuda", dtype=torch.int32)
    elif ragged:
        ln = torch.randint(T // 8, T + 1, (n,), generator=g, device="cuda", dtype=torch.int32)
        ln[0], ln[-1] = T, 0
    pad = torch.arange(T, device="cuda").repeat(n) >= (T if ln is None else ln.repeat_interleave(T))

    def rows(d, scale=1.0):
        x = (rand(n * T, d) * scale).to(dtype)
        x[pad] = float("nan")
        return x
    mods = []
    for _ in range(layers):
        seen = {}
        for a, b, tag in layer:
            seen.setdefault(tag, rows(a))
            mods.append(P.Module(seen[tag] if shared else seen[tag].clone(), rows(b, 1e-2),
                                 (rand(b, k) / k ** 0.5).to(dtype), (rand(a, k) / k ** 0.5).to(dtype),
                                 len(mods) * k * k))
    return mods, ln


def exact(m, n, T, ln):
    """[n, T, k] projected rows of a module in fp64, zeros past the lengths."""
    x, y = m.g.double() @ m.R.double(), m.a.double() @ m.S.double()
    x, y = (torch.nan_to_num(z).reshape(n, T, -1) for z in (x, y))
    return x, y


def check_rows(out, mods, dt, k, n, T, ln):
    bar = 1e-5 if dt == "f32" else 1e-4
    for m in mods:
        x, y = exact(m, n, T, ln)
        ref = torch.bmm(x.transpose(1, 2).contiguous(), y).reshape(n, k * k)
        got = out[:, m.out_col:m.out_col + k * k].double()
        some = ref.norm(dim=1) > 0
        assert (got[~some] == 0).all() and (ln is None or (~some).sum() == (ln == 0).sum())
        assert ((got - ref).norm(dim=1)[some] <= bar * ref.norm(dim=1)[some]).all()


def check_tokens(out, rows, mods, dt, k, n, T, ln):
    """out: the blocks of token rows [0, rows), and rows that the call must not touch."""
    pad = torch.zeros(n * T, dtype=torch.bool, device="cuda")
    if ln is not None:
        pad = torch.arange(T, device="cuda").repeat(n) >= ln.repeat_interleave(T)
    written = torch.zeros(out.shape[0], dtype=torch.bool, device="cuda")
    written[:rows] = ~pad[:rows]
    assert (out[~written] == 7.0).all()
    bar = 1e-5 if dt == "f32" else 1e-4
    for m in mods:
        x, y = (z.reshape(n * T, k)[written[:n * T]] for z in exact(m, n, T, ln))
        got = out[written, m.out_col:m.out_col + k * k].reshape(-1, k, k)
        for i in range(0, got.shape[0], 8192):
            ref = x[i:i + 8192, :, None] * y[i:i + 8192, None, :]
            err = (got[i:i + 8192].double() - ref).flatten(1).norm(dim=1)
            assert (err <= bar * ref.flatten(1).norm(dim=1)).all()


@pytest.mark.parametrize("dt,k,layers,n,T,ragged,route", ROUTES)
def test_shared_rows_give_the_bits_of_separate_copies(dt, k, layers, n, T, ragged, route):
    say(f"case: {dt} k={k} {layers} layers {n} x {T} lengths={ragged} ({route})")
    out = []
    for shared in (True, False):
        mods, ln = make(dt, k, layers, n, T, ragged, shared)
        out.append(torch.full((n, len(mods) * k * k), 7.0, device="cuda"))
        P.attr_project(mods, k, n, T, out[-1], length=ln)
    assert torch.equal(out[0], out[1])
    check_rows(out[0], mods, dt, k, n, T, ln)


@pytest.mark.parametrize("dt,k,layers,n,T,ragged,route", TOKEN_ROUTES)
def test_token_blocks(dt, k, layers, n, T, ragged, route):
    say(f"case: per token {dt} k={k} {layers} layers {n} x {T} lengths={ragged} ({route})")
    mods, ln = make(dt, k, layers, n, T, ragged)
    rows = n * T - 5  # the last rows are past the output
    out = torch.full((rows + 5, len(mods) * k * k), 7.0, device="cuda")
    P.attr_project_tokens(mods, k, n, T, out[:rows], length=ln)
    check_tokens(out, rows, mods, dt, k, n, T, ln)


@pytest.mark.parametrize("dt", ["bf16", "f32"])
@pytest.mark.parametrize("k", [16, 32, 64])
@pytest.mark.parametrize("shapes,n,T,lengths", WIDE)
def test_few_tokens_of_wide_modules(dt, k, shapes, n, T, lengths):
    say(f"case: wide {dt} k={k} {shapes} {n} x {T} lengths={lengths}")
    layer = [(a, b, j) for j, (a, b) in enumerate(shapes)]
    mods, ln = make(dt, k, 1, n, T, False, layer=layer, lengths=lengths)
    out = torch.full((n, len(mods) * k * k), 7.0, device="cuda")
    P.attr_project(mods, k, n, T, out, length=ln)
    check_rows(out, mods, dt, k, n, T, ln)
    rows = n * T
    tok = torch.full((rows + 3, len(mods) * k * k), 7.0, device="cuda")
    P.attr_project_tokens(mods, k, n, T, tok[:rows], length=ln)
    check_tokens(tok, rows, mods, dt, k, n, T, ln)
