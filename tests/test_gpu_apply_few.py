"""GPU: the FULL apply on few rows (M read once, split on the way), against fp64.

The bound per element follows from the arithmetic: M's two fp16 halves hold
it to 2^-22, products are exact in fp32, and each of the D / 32 matrix-core
steps of either half (and each slice sum) rounds the running sum once, so
|y - ref| <= (2^-22 + (2 D / 32 + 16) 2^-23) sum_q |M_pq x_q|.
"""
import pytest
import torch

import paper_2606_11660_amd as P

pytestmark = pytest.mark.gpu


def _case(n, D, seed, ldx=None):
    g = torch.Generator(device="cuda")
    g.manual_seed(seed)
    buf = torch.full((n, ldx or D), float("nan"), dtype=torch.float16, device="cuda")
    X = buf[:, :D]
    X.copy_(torch.randn((n, D), generator=g, device="cuda"))
    return X, torch.randn((D, D), generator=g, device="cuda") / D ** 0.5


def _bound(X, M):
    return (2.0 ** -22 + (M.shape[0] / 16 + 16) * 2.0 ** -23) * (X.double().abs() @ M.double().abs().T)


# rows: one, the edges of the 16-row tiles and of the 64 / 128 / 256-row
# workgroups, several row blocks; D: one stage, ragged stage groups, several
# K-slices, the largest row count of the path
@pytest.mark.parametrize("n,D", [(1, 64), (64, 64), (15, 128), (16, 320), (17, 320), (64, 1024),
                                 (65, 1088), (128, 576), (129, 576), (256, 2048), (257, 2048),
                                 (1000, 1024), (1024, 8192)])
@pytest.mark.parametrize("scale", ["one", "rows", "grow", "fall"])
def test_apply_few_unscaled(n, D, scale):
    if D == 8192 and scale != "one":
        pytest.skip("large case once")
    X, M = _case(n, D, 1, ldx=D + 64)
    if scale == "rows":      # rows of M far apart, some all zero
        M *= torch.logspace(-18, 18, D, device="cuda")[:, None]
        M[::7] = 0
    elif scale == "grow":    # the running exponent moves at every stage
        M *= torch.logspace(-9, 3, D, device="cuda")[None, :]
        M[:, : D // 4] = 0
    elif scale == "fall":
        M *= torch.logspace(3, -9, D, device="cuda")[None, :]
    M = M.contiguous()
    Y = torch.empty((n, D), device="cuda")
    P.attr_precond_apply(X, P.PRECOND_FULL, M, False, Y)
    ref = X.double() @ M.double().T
    over = (Y.double() - ref).abs() - _bound(X, M)
    assert over.max().item() <= 0.0
    Z = torch.empty_like(Y)
    P.attr_precond_apply(X, P.PRECOND_FULL, M, False, Z)
    assert torch.equal(Y, Z)


@pytest.mark.parametrize("n,D", [(3, 64), (100, 1088), (300, 8256)])
@pytest.mark.parametrize("dtype", [torch.float16, torch.float32])
def test_apply_few_unit(n, D, dtype):
    X, M = _case(n, D, 2)
    M *= 300.0  # un-normalised rows pass fp16's range at some entries
    X[0] = 0
    wide = torch.full((n, D + 32), 7.0, dtype=dtype, device="cuda")
    Y = wide[:, :D]
    P.attr_precond_apply(X, P.PRECOND_FULL, M, True, Y)
    ref = X.double() @ M.double().T
    norm = ref.norm(dim=1, keepdim=True)
    err = (Y.double() - torch.where(norm > 0, ref / norm, 0.0)).norm(dim=1)
    tol = _bound(X, M).norm(dim=1) / norm[:, 0].clamp(min=1e-30) + 2.0 ** (-11 if dtype == torch.float16 else -23)
    assert (err[1:] <= tol[1:]).all() and err[0] == 0
    assert (wide[:, D:] == 7.0).all()


def test_apply_few_nan_stays_in_its_column():
    X, M = _case(40, 512, 3)
    M[77, 100] = float("nan")
    Y = torch.empty((40, 512), device="cuda")
    P.attr_precond_apply(X, P.PRECOND_FULL, M, False, Y)
    bad = torch.isnan(Y)
    assert bad[:, 77].all() and bad.sum().item() == 40


@pytest.mark.parametrize("dtype", [torch.float16, torch.float32])
def test_rows_with_nan_are_those_of_the_general_path(dtype):
    """unit rows: a NaN stays where it is and the row is zero elsewhere, in a call of
    few rows as in one of more than D rows (the general path)."""
    X, M = _case(520, 512, 4)
    X[3] = float("nan")
    M[77, 100] = float("nan")
    few, many = (torch.full((n, 512), 7.0, dtype=dtype, device="cuda") for n in (40, 520))
    P.attr_precond_apply(X[:40], P.PRECOND_FULL, M, True, few)
    P.attr_precond_apply(X, P.PRECOND_FULL, M, True, many)
    for Y in (few, many):
        bad = torch.isnan(Y)
        assert bad[3].all() and bad[:, 77].all() and bad.sum() == 512 + Y.shape[0] - 1
        assert (Y[~bad] == 0).all()
