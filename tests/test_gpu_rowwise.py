"""The wide-row normaliser (more than 8192 columns: one or two rows per workgroup, 512
or 1024 threads, three or four chunks each) and the column sums at the edges of
their layouts: widths one chunk past and at each limit, odd row counts, in place,
with and without scale and norm.  Bars: one fp16 ulp (2^-11 relative, plus half a
subnormal) for fp16 rows; 1e-6 relative for fp32 rows (a norm of D fp32 squares in
chains of at most 64: 64 2^-24 / 2 = 2e-6 of the square, 1e-6 of the norm) and for
the column sums, as the accumulate's own test."""
import numpy as np
import pytest
import torch

import paper_2606_11660_amd as P
from tests._util import say

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("D", [8192, 8200, 12288, 12296, 16384, 16392, 24576, 24584, 32768, 32776])
@pytest.mark.parametrize("dtype", [torch.float16, torch.float32])
@pytest.mark.parametrize("n", [1, 7])
def test_wide_rows(D, dtype, n):
    say(f"case: wide rows D={D} n={n} {dtype}")
    g = torch.Generator(device="cuda").manual_seed(D + n)
    X = torch.randn((n, D + 8), generator=g, device="cuda").to(dtype)[:, :D]
    X[n // 2] = 0
    m = torch.rand(D, generator=g, device="cuda") + 0.5
    for mode, scale in ((P.PRECOND_DIAG, m), (P.PRECOND_NONE, None)):
        for unit in (True, False):
            x = X.double() * (scale.double() if scale is not None else 1.0)
            if unit:
                x = x / x.norm(dim=1, keepdim=True).clamp_min(1e-300)
            for yd, rel, sub in ((torch.float16, 2.0 ** -11, 2.0 ** -25), (torch.float32, 1e-6, 0.0)):
                Y = torch.full((n, D + 16), 9.0, dtype=yd, device="cuda")
                P.attr_precond_apply(X, mode, scale, unit, Y[:, :D])
                err = (Y[:, :D].double() - x).abs()
                assert (err <= 1.01 * rel * x.abs() + sub).all(), (mode, unit, yd, err.max().item())
                assert (Y[:, D:] == 9.0).all()
            Z = X.contiguous().clone()
            P.attr_precond_apply(Z, mode, scale, unit, Z)
            Y = torch.empty_like(Z)
            P.attr_precond_apply(X, mode, scale, unit, Y)
            assert torch.equal(Z, Y)


@pytest.mark.parametrize("xd,yd,D,n", [
    (torch.float16, torch.float16, 8200, 513), (torch.float16, torch.float16, 16384, 512),
    (torch.float16, torch.float16, 24576, 257), (torch.float16, torch.float32, 12288, 10001),
    (torch.float16, torch.float32, 24584, 300), (torch.float32, torch.float16, 16384, 8193),
    (torch.float32, torch.float16, 24576, 1025), (torch.float32, torch.float16, 32768, 1025)])
def test_wide_rows_alone_and_among_many(xd, yd, D, n):
    """One and two rows per workgroup (few and many rows) give a row the same bits."""
    say(f"case: wide rows {n} x {D} {xd} to {yd}")
    g = torch.Generator(device="cuda").manual_seed(D + n)
    X = torch.randn((n, D), generator=g, device="cuda").to(xd)
    m = torch.rand(D, generator=g, device="cuda") + 0.5
    for mode, scale in ((P.PRECOND_DIAG, m), (P.PRECOND_NONE, None)):
        Y = torch.empty((n, D), dtype=yd, device="cuda")
        P.attr_precond_apply(X, mode, scale, True, Y)
        few = torch.empty((3, D), dtype=yd, device="cuda")
        P.attr_precond_apply(X[-3:], mode, scale, True, few)
        assert torch.equal(Y[-3:], few)
        x = X[-99:].double() * (scale.double() if scale is not None else 1.0)
        x = x / x.norm(dim=1, keepdim=True)
        rel, sub = (2.0 ** -11, 2.0 ** -25) if yd == torch.float16 else (1e-6, 0.0)
        assert ((Y[-99:].double() - x).abs() <= 1.01 * rel * x.abs() + sub).all()


@pytest.mark.parametrize("dtype", [torch.float32, torch.float16, torch.bfloat16])
@pytest.mark.parametrize("n,D", [(1, 8), (7, 1024), (9, 1032), (64, 2056), (1000, 1000), (40000, 128), (70001, 72)])
def test_column_sums(n, D, dtype):
    say(f"case: column sums n={n} D={D} {dtype}")
    g = torch.Generator(device="cuda").manual_seed(n)
    X = torch.randn((n, D + 16), generator=g, device="cuda").to(dtype)
    X[:, D:] = float("nan")
    X = X[:, :D]
    h = torch.rand(D, generator=g, device="cuda")
    want = h.double() + X.double().square().sum(0)
    P.attr_precond_accumulate(X, P.PRECOND_DIAG, h)
    assert ((h.double() - want).abs() <= 1e-6 * want).all()
