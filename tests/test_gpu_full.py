"""GPU parity of the full second-moment preconditioner: attr_precond_accumulate
(FULL, H += X^T X) and attr_precond_apply (FULL, y = M x, unit norm)."""
import numpy as np
import pytest
import torch

import oracle as O
import paper_2606_11660_amd as P
from paper_2606_11660_amd import finalize as fin
import synth
from tests._util import dev, host, row_rel_l2, say

pytestmark = pytest.mark.gpu


def _syrk(X, H0=None, chunks=None):
    D = X.shape[1]
    if H0 is None:
        H = torch.full((D, D), 7.0, dtype=torch.float32, device="cuda")
        H[torch.triu(torch.ones(D, D, dtype=torch.bool, device="cuda"))] = 0.0
    else:
        H = H0
    Xd = dev(X) if isinstance(X, np.ndarray) else X
    if chunks is None:
        P.attr_precond_accumulate(Xd, P.PRECOND_FULL, H)
    else:
        for lo, hi in chunks:
            P.attr_precond_accumulate(Xd[lo:hi], P.PRECOND_FULL, H)
    torch.cuda.synchronize()
    return host(H)


def _check_upper(got, ref, tol=1e-5):
    iu = np.triu_indices(ref.shape[0])
    err = np.abs(got[iu] - ref[iu]).max() / np.abs(ref).max()
    il = np.tril_indices(ref.shape[0], -1)
    assert (got[il] == 7.0).all(), "strict lower triangle was written"
    return err


@pytest.mark.parametrize("n,D", [(3000, 512), (777, 320), (70001, 256), (263144, 256)])
def test_syrk_matches_oracle(n, D):
    say(f"case: syrk n={n} D={D}")
    X = (np.random.default_rng(n).standard_normal((n, D)) * 2).astype(np.float16)
    got = _syrk(X)
    err = _check_upper(got, O.accumulate_full(X))
    say("max rel err", err)
    assert err <= 1e-5


@pytest.mark.parametrize("n", [1, 63, 64, 65, 128, 129, 192, 200, 320, 449])
def test_syrk_short_slices(n):
    """Row counts whose slices hold one to a few K-stages (ragged last stage;
    odd and even stage counts reach both ends of the stage loop)."""
    say(f"case: syrk short n={n} D=256")
    X = (np.random.default_rng(1000 + n).standard_normal((n, 256)) * 2).astype(np.float16)
    err = _check_upper(_syrk(X), O.accumulate_full(X))
    say("max rel err", err)
    assert err <= 1e-5


def test_kfac_factors_from_packed_token_rows():
    """K-FAC factors (A = sum a a^T, Gamma = sum g g^T over the valid tokens)
    of two modules of a ragged batch: each is the FULL accumulate of the
    module's token rows packed back to back (bf16); compared with the
    oracle's factors of the padded batch.  The 2048-wide case has few
    upper tiles, so the accumulate splits its rows into more slices."""
    rng = np.random.default_rng(71)
    n, T = 4, 1200
    lengths = [300, 17, 1200, 512]
    mods = [(256, 512), (2048, 128)]
    say("case: K-FAC factors from packed token rows")
    for d_in, d_out in mods:
        a = synth.to_bf16_bits(rng.standard_normal((n, T, d_in)))
        g = synth.to_bf16_bits(rng.standard_normal((n, T, d_out)))
        a_pk = np.concatenate([a[i, :lengths[i]] for i in range(n)])
        g_pk = np.concatenate([g[i, :lengths[i]] for i in range(n)])
        an = np.stack([synth.nan_pad(a[i], lengths[i]) for i in range(n)])
        gn = np.stack([synth.nan_pad(g[i], lengths[i]) for i in range(n)])
        A, Gm = O.kfac_factors(an, gn, length=lengths)
        for X, ref in ((a_pk, A), (g_pk, Gm)):
            Xt = torch.from_numpy(X.view(np.int16)).view(torch.bfloat16).cuda()
            err = _check_upper(_syrk(Xt), ref)
            say(f"d={ref.shape[0]} max rel err {err:.2e}")
            assert err <= 1e-5


def test_syrk_additive_bf16_and_chunks():
    say("case: syrk additive over calls, bf16")
    n, D = 5000, 384
    Xf = np.random.default_rng(1).standard_normal((n, D))
    bits = synth.to_bf16_bits(Xf)
    Xt = torch.from_numpy(bits.view(np.int16)).view(torch.bfloat16).cuda()
    got = _syrk(Xt, chunks=[(0, 1234), (1234, 5000)])
    err = _check_upper(got, O.accumulate_full(bits))
    say("max rel err", err)
    assert err <= 1e-5


def test_syrk_lowrank_small_eigenvalues():
    """Low-rank-plus-noise store (rank 64, noise 0.1): the noise eigenvalues of
    H / N sit ~6 decades below the signal ones; the GPU H must keep them to 1%."""
    say("case: syrk low-rank spectrum")
    D, N = 1024, 60000
    X = synth.lowrank_rows(0, N, D=D, rank=64, chunk=16384)
    got = _syrk(X)
    ref = O.accumulate_full(X)
    Hs = np.triu(got.astype(np.float64))
    Hs = (Hs + np.triu(Hs, 1).T) / N
    lam_g = np.sort(np.linalg.eigvalsh(Hs))
    lam_r = np.sort(np.linalg.eigvalsh(ref / N))
    small = slice(0, D - 64)
    rel = np.abs(lam_g[small] - lam_r[small]) / lam_r[small]
    say("small-eigenvalue max rel err", rel.max(), "kappa", lam_r[-1] / lam_r[0])
    assert rel.max() <= 1e-2


@pytest.mark.parametrize("n,D", [(1000, 512), (777, 320), (300, 64)])
def test_full_apply_well_conditioned(n, D):
    """Random SPD M; ragged row tiles (777 = 3 x 256 + 9, 300 = 256 + 44), a
    ragged 64-column tile and an odd count of 64-wide K-blocks (D = 320:
    the hi/lo-interleaved core's last pair of steps), a single K-block
    (D = 64)."""
    say(f"case: full apply, random SPD M n={n} D={D}")
    rng = np.random.default_rng(3)
    X = (rng.standard_normal((n, D)) * 3).astype(np.float16)
    B = rng.standard_normal((D, D)) / np.sqrt(D)
    M = (B @ B.T + 0.5 * np.eye(D)).astype(np.float32)
    for unit in (False, True):
        for ydt in (torch.float32, torch.float16):
            Y = torch.empty((n, D), dtype=ydt, device="cuda")
            P.attr_precond_apply(dev(X), P.PRECOND_FULL, dev(M), unit, Y)
            torch.cuda.synchronize()
            ref = O.precond_apply(X, "full", M.astype(np.float64), unit_norm=unit)
            err = row_rel_l2(host(Y), ref)
            say(f"unit={unit} y={ydt} max row rel-L2 {err.max():.2e}")
            assert err.max() <= (1e-5 if ydt == torch.float32 else 2e-3)


def test_preconditioner_pipeline_lowrank():
    """Reduced precond workload: accumulate H on the GPU, finalize on the host,
    apply H^{-1/2} + unit norm on the GPU to store rows and queries; compare
    with the oracle pipeline built on the exact H."""
    say("case: full preconditioner pipeline, low-rank store")
    D, N, nq = 1024, 40000, 64
    F = synth.lowrank_factor(D, 64, seed=3)
    X = synth.lowrank_rows(0, N, D=D, rank=64, chunk=16384, F=F)
    Qh = synth.lowrank_queries(nq, D=D, rank=64, F=F)
    Xd, Qd = dev(X), dev(Qh)
    H = torch.zeros((D, D), dtype=torch.float32, device="cuda")
    P.attr_precond_accumulate(Xd, P.PRECOND_FULL, H)
    M = fin.finalize_full(H, N)
    Y = torch.empty((N, D), dtype=torch.float16, device="cuda")
    YQ = torch.empty((nq, D), dtype=torch.float16, device="cuda")
    P.attr_precond_apply(Xd, P.PRECOND_FULL, M, True, Y)
    P.attr_precond_apply(Qd, P.PRECOND_FULL, M, True, YQ)
    torch.cuda.synchronize()
    Mr, lam = O.finalize_full(O.accumulate_full(X), N)
    sample = np.arange(0, N, 97)
    ref = O.precond_apply(X[sample], "full", Mr, unit_norm=True)
    err = row_rel_l2(host(Y)[sample], ref)
    refq = O.precond_apply(Qh, "full", Mr, unit_norm=True)
    errq = row_rel_l2(host(YQ), refq)
    say(f"store rows max rel-L2 {err.max():.2e}, queries {errq.max():.2e}, kappa {lam.max() / lam.min():.2e}")
    assert err.max() <= 2e-2 and errq.max() <= 2e-2
    assert np.abs(np.linalg.norm(host(Y)[sample].astype(np.float64), axis=1) - 1).max() <= 2e-3


def test_full_apply_unit_rows_beyond_fp16_range():
    """Rows whose whitened, un-normalised values exceed fp16's range (a large
    component along the eigenvector of the smallest kept eigenvalue, which
    H^{-1/2} amplifies most) and rows whose values sit far below fp16's
    normal range: the unit rows written as fp16 are still finite and match
    the oracle, on both the fp16 and the fp32 output paths."""
    say("case: full apply, rows beyond fp16 range")
    D, N = 512, 20000
    F = synth.lowrank_factor(D, 64, seed=3)
    X = synth.lowrank_rows(0, N, D=D, rank=64, chunk=8192, F=F)
    M, lam = O.finalize_full(O.accumulate_full(X), N)
    _, V = np.linalg.eigh(O.accumulate_full(X) / N)
    v = V[:, 0] / np.abs(V[:, 0]).max()                 # smallest eigenvalue's direction
    rng = np.random.default_rng(5)
    rows = [30000.0 * v,                                 # |M x| ~ 3e5: past 65504
            30000.0 * v + 100.0 * rng.standard_normal(D),
            -20000.0 * v,
            5e-7 * rng.standard_normal(D),               # |M x| < 6.1e-5: fp16 subnormals
            X[7].astype(np.float64)]                     # an ordinary store row
    Q = np.stack(rows).astype(np.float16)
    Md = dev(M.astype(np.float32))
    ref = O.precond_apply(Q, "full", M.astype(np.float32).astype(np.float64), unit_norm=True)
    raw = O.precond_apply(Q, "full", M.astype(np.float32).astype(np.float64), unit_norm=False)
    assert np.abs(raw[:3]).max(axis=1).min() > 65504 and np.abs(raw[3]).max() < 6.1e-5
    for ydt in (torch.float16, torch.float32):
        Y = torch.empty((Q.shape[0], D), dtype=ydt, device="cuda")
        P.attr_precond_apply(dev(Q), P.PRECOND_FULL, Md, True, Y)
        torch.cuda.synchronize()
        got = host(Y).astype(np.float64)
        assert np.isfinite(got).all(), f"{ydt}: non-finite unit rows"
        err = row_rel_l2(got, ref)
        say(f"y={ydt} max row rel-L2 {err.max():.2e}")
        assert err.max() <= 2e-3


@pytest.mark.parametrize("ydt", [torch.float16, torch.float32])
def test_full_apply_beyond_fp16_range_in_a_call_of_many_rows(ydt):
    """The rows of the test above in a call of more rows than D, which takes the
    general path: with an fp16 Y its intermediate is fp16, scaled per 128-column
    segment by an exponent that the second pass takes back."""
    say("case: full apply, rows beyond fp16 range among many")
    D, N = 512, 20000
    F = synth.lowrank_factor(D, 64, seed=3)
    X = synth.lowrank_rows(0, N, D=D, rank=64, chunk=8192, F=F)
    M, lam = O.finalize_full(O.accumulate_full(X), N)
    _, V = np.linalg.eigh(O.accumulate_full(X) / N)
    v = V[:, 0] / np.abs(V[:, 0]).max()
    rng = np.random.default_rng(5)
    far = np.stack([30000.0 * v, 30000.0 * v + 100.0 * rng.standard_normal(D), -20000.0 * v,
                    5e-7 * rng.standard_normal(D)]).astype(np.float16)
    Q = np.concatenate([far, X[:D].astype(np.float16), far])
    M32 = M.astype(np.float32)
    ref = O.precond_apply(Q, "full", M32.astype(np.float64), unit_norm=True)
    raw = O.precond_apply(far, "full", M32.astype(np.float64), unit_norm=False)
    assert np.abs(raw[:3]).max(axis=1).min() > 65504 and np.abs(raw[3]).max() < 6.1e-5
    Y = torch.empty((Q.shape[0], D), dtype=ydt, device="cuda")
    P.attr_precond_apply(dev(Q), P.PRECOND_FULL, dev(M32), True, Y)
    torch.cuda.synchronize()
    got = host(Y).astype(np.float64)
    assert np.isfinite(got).all()
    err = row_rel_l2(got, ref)
    say(f"y={ydt} max row rel-L2 {err.max():.2e}")
    assert err.max() <= 2e-3
