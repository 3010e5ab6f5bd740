"""Canonical <-> packed conversion at the edges of its blocks (128 and 256
checkerboard sites) and from pointers aligned to a double only.

Small lattices read and write the canonical field in the hop itself; WL_TUNE=0
takes them through the packed fields as larger ones are, so both routes are run.

With parity -1 and kappa = 0 a D-slash call packs its input and unpacks the
epilogue's 1 * x + 0, so the output is the storage rounding of the input, bit for
bit (the host model of tests/gpu_util.py; exact in FP64).  A single-parity hop
must equal the parity of the whole operator's hop and zeros elsewhere.
"""
import numpy as np
import pytest

import lattice_inputs as li
import oracle
from tests.gpu_util import need_gpu, quantize_spinor, to_dev

pytestmark = pytest.mark.gpu

# sites per parity: 8 (less than a wave), 120, 128, 264, 256, 528, 840
SHAPES = [(2, 2, 2, 2), (2, 6, 2, 10), (4, 4, 4, 4), (2, 2, 6, 22), (4, 4, 4, 8), (4, 2, 6, 22), (2, 10, 6, 14)]


@pytest.mark.parametrize("L", SHAPES)
@pytest.mark.parametrize("prec", ["f64", "f32", "f16", "bf16"])
@pytest.mark.parametrize("offset", [0, 1])
@pytest.mark.parametrize("tune", ["1", "0"])
def test_round_trip(L, prec, offset, tune, monkeypatch):
    w = need_gpu()
    monkeypatch.setenv("WL_TUNE", tune)
    import torch

    nrhs = 2
    psi = li.gaussian_spinor(L, 11, nrhs=nrhs)
    n = psi.size * 2
    inp = torch.zeros(n + 1, dtype=torch.float64, device="cuda")[offset:offset + n]
    out = torch.full((n + 3,), float("nan"), dtype=torch.float64, device="cuda")
    inp.copy_(torch.from_numpy(psi.view(np.float64).reshape(-1)))
    o = out[offset + 1:offset + 1 + n]
    g = w.Gauge(L, to_dev(li.haar_links(L, 12)))
    w.wilson_dslash(g, inp, o, nrhs, 0.0, -1, 0, prec, 12)
    got = o.cpu().numpy()
    want = psi.astype(np.complex64).astype(np.complex128) if prec == "f32" else psi
    want = quantize_spinor(psi, prec) if prec in ("f16", "bf16") else want
    assert np.array_equal(got, want.view(np.float64).reshape(-1))
    whole = out.cpu().numpy()  # nothing written outside the field
    assert np.isnan(np.delete(whole, np.s_[offset + 1:offset + 1 + n])).all()
    g.close()


@pytest.mark.parametrize("L", SHAPES)
@pytest.mark.parametrize("parity", [0, 1])
@pytest.mark.parametrize("tune", ["1", "0"])
def test_other_parity_is_zero(L, parity, tune, monkeypatch):
    w = need_gpu()
    monkeypatch.setenv("WL_TUNE", tune)
    import torch

    U, psi = li.haar_links(L, 13), li.gaussian_spinor(L, 14, nrhs=3)
    g = w.Gauge(L, to_dev(U))
    out = torch.full((psi.size * 2,), float("nan"), dtype=torch.float64, device="cuda")
    w.wilson_dslash(g, to_dev(psi), out, 3, 0.0, parity, 0, "f64", 18)
    got = out.cpu().numpy().view(np.complex128).reshape(psi.shape)
    ref = oracle.hop(L, U, psi, out_parity=parity)
    assert np.array_equal(got == 0, ref == 0)
    assert np.abs(got - ref).max() <= 1e-13 * np.abs(ref).max() * 8  # 8 directions of FP64 products
    g.close()


@pytest.mark.parametrize("L", [(2, 2, 2, 2), (4, 4, 4, 2), (2, 10, 6, 14)])
@pytest.mark.parametrize("prec", ["f64", "f32", "f16", "bf16"])
@pytest.mark.parametrize("csw", [None, 1.3])
def test_routes_agree(L, prec, csw, monkeypatch):
    """The canonical field read in the hop and the packed one give the same bits."""
    w = need_gpu()
    U, psi = li.haar_links(L, 15), li.gaussian_spinor(L, 16, nrhs=3)
    psi[1] = 0
    for parity, dagger in [(-1, 0), (-1, 1)] + ([(0, 1), (1, 0)] if csw is None else []):
        out = []
        for tune in ("1", "0"):
            monkeypatch.setenv("WL_TUNE", tune)
            g = w.Gauge(L, to_dev(U))
            o = to_dev(np.full_like(psi, np.nan))
            if csw is None:
                w.wilson_dslash(g, to_dev(psi), o, 3, 0.13, parity, dagger, prec, 12)
            else:
                w.wilson_clover_dslash(g, to_dev(psi), o, 3, 0.13, csw, dagger, prec, 12)
            out.append(o.cpu().numpy())
            g.close()
        assert np.array_equal(out[0], out[1]), (parity, dagger)


@pytest.mark.parametrize("L", SHAPES)
@pytest.mark.parametrize("prec", ["f64", "f32", "f16", "bf16"])
@pytest.mark.parametrize("parity", [-1, 0, 1])
def test_unpack(L, prec, parity):
    """The unpacking kernels, which wilson_dslash_noalloc still uses, on pointers
    aligned to a double: both parities of a packed field with kappa = 0 (the input as
    storage leaves it), or one parity, as the call that stores the canonical field in
    the hop gives it, and zeros on the other."""
    w = need_gpu()
    import torch

    nrhs = 2
    psi = li.gaussian_spinor(L, 17, nrhs=nrhs)
    n = psi.size * 2
    inp = torch.zeros(n + 1, dtype=torch.float64, device="cuda")[1:]
    out = torch.full((n + 3,), float("nan"), dtype=torch.float64, device="cuda")
    ref = torch.full((n,), float("nan"), dtype=torch.float64, device="cuda")
    inp.copy_(torch.from_numpy(psi.view(np.float64).reshape(-1)))
    g = w.Gauge(L, to_dev(li.haar_links(L, 18)))
    w.wilson_dslash_noalloc(g, inp, out[1:1 + n], nrhs, 0.0, parity, 0, prec, 12)
    w.wilson_dslash(g, inp, ref, nrhs, 0.0, parity, 0, prec, 12)
    got, want = out.cpu().numpy(), ref.cpu().numpy()
    assert np.array_equal(got[1:1 + n], want)
    if parity < 0:
        q = psi.astype(np.complex64).astype(np.complex128) if prec == "f32" else psi
        q = quantize_spinor(psi, prec) if prec in ("f16", "bf16") else q
        assert np.array_equal(want, q.view(np.float64).reshape(-1))
    assert np.isnan(got[0]) and np.isnan(got[1 + n:]).all()  # nothing written outside the field
    g.close()
