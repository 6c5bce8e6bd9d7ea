"""The native gatherer of module descriptors against the binding's Python
checks: the same descriptors for every form that it accepts, None (so that the
Python checks decide) for what it does not."""
import pytest
import torch

import paper_2606_11660_amd as P

pytestmark = pytest.mark.gpu


def _call(n=3, T=5, k=16, dtype=torch.bfloat16, lead=False, wide=0, factors=False, rows=15, mods=2):
    dev = "cuda"
    out = torch.zeros((n, mods * k * k + 8), device=dev)
    ms = []
    for j in range(mods):
        a, g = (torch.zeros((rows, w + wide), dtype=dtype, device=dev)[:, :w] for w in (64, 128))
        if lead:
            a, g = a.unflatten(0, (n, T)), g.unflatten(0, (n, T))
        v = dict(v_out=torch.ones(128, device=dev), v_in=torch.ones(64, device=dev)) if factors and j else {}
        ms.append(P.Module(a, g, torch.zeros((128, k), dtype=dtype, device=dev),
                           torch.zeros((64, k), dtype=dtype, device=dev), j * k * k, **v))
    return [ms, k, n, T, None, None, out, n]


def _native(c):
    return P._native()(c[0], P.Module, *c[1:])


@pytest.mark.parametrize("kw", [{}, dict(dtype=torch.float32, k=32), dict(lead=True), dict(wide=64),
                                dict(factors=True), dict(lead=True, wide=8, factors=True, mods=5), dict(n=0)])
def test_descriptors_equal_the_python_ones(kw):
    c = _call(**kw)
    for mods in (c[0], tuple(c[0])):
        code, buf = _native([mods] + c[1:])
        assert code == P._check_modules(*c)
        assert bytes(buf) == bytes(P._cmods(c[0]))
    off, ln = torch.zeros(c[2], dtype=torch.int64, device="cuda"), torch.ones(c[2], dtype=torch.int32, device="cuda")
    c[4], c[5] = off, ln
    assert bytes(_native(c)[1]) == bytes(P._cmods(c[0]))


def _break(name):
    c = _call()
    m = c[0][1]
    if name == "cpu":
        m.a = m.a.cpu()
    elif name == "dtype":
        m.g = m.g.float()
    elif name == "last stride":
        m.a = torch.zeros((64, 15), dtype=m.a.dtype, device="cuda").t()
    elif name == "leading stride":
        m.a = torch.zeros((3, 7, 64), dtype=m.a.dtype, device="cuda")[:, :5]
    elif name == "R strided":
        m.R = torch.zeros((16, 128), dtype=m.R.dtype, device="cuda").t()
    elif name == "S shape":
        m.S = m.R
    elif name == "rows":
        m.g = m.g[:14]
    elif name == "factor":
        m.v_out, m.v_in = torch.ones(127, device="cuda"), torch.ones(64, device="cuda")
    elif name == "column":
        m.out_col = 257 + 8
    elif name == "out rows":
        c[7] = 4
    elif name == "offsets":
        c[4] = torch.zeros(2, dtype=torch.int64, device="cuda")
    elif name == "lengths":
        c[5] = torch.zeros(3, dtype=torch.int64, device="cuda")
    elif name == "T":
        c[3] = 0
    elif name == "none":
        c[0] = []
    return c


@pytest.mark.parametrize("name", ["cpu", "dtype", "last stride", "leading stride", "R strided", "S shape", "rows",
                                  "factor", "column", "out rows", "offsets", "lengths", "T", "none"])
def test_what_the_python_checks_refuse_is_left_to_them(name):
    c = _break(name)
    assert _native(c) is None
    with pytest.raises(ValueError):
        P._check_modules(*c)
        P._cmods(c[0])


def test_other_kinds_are_left_to_the_python_checks():
    class Sub(torch.Tensor):
        pass

    class Mod(P.Module):
        pass
    c = _call()
    c[0][0].a = c[0][0].a.as_subclass(Sub)
    assert _native(c) is None and P._check_modules(*c) == P.ATTR_BF16
    c = _call()
    c[0][0].__class__ = Mod
    assert _native(c) is None and P._check_modules(*c) == P.ATTR_BF16
