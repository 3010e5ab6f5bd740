"""The hop variant that puts the eight directions of 64 sites on eight waves, against
the per-site variant 3: the same D-slash bit for bit (whole and partial blocks of
64 sites, several right-hand sides, both parities in one launch and alone), and
solves through its reductions (|out|^2, <X1, out>, <out, X0>)."""
import numpy as np
import pytest

import lattice_inputs as li
import oracle
from tests.gpu_util import from_dev, need_gpu, to_dev
from tests.test_gpu_dslash import CASES, run_dslash

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("L", [(2, 2, 2, 2), (4, 4, 4, 2), (4, 6, 2, 8), (2, 10, 6, 14)])  # 8, 64, 192, 840 sites a parity
@pytest.mark.parametrize("prec,recon", CASES)
def test_split_equals_per_site(L, prec, recon, monkeypatch):
    w = need_gpu()
    U, psi = li.haar_links(L, 61), li.gaussian_spinor(L, 62, nrhs=3)
    for parity, dagger in [(0, 0), (1, 1), (-1, 0), (-1, 1)]:
        out = []
        for cfg in ("3:256", "11:64"):
            monkeypatch.setenv("WL_TUNE_FORCE", cfg)
            out.append(run_dslash(w, L, U, psi, 0.13, parity, dagger, prec, recon))
        assert np.array_equal(out[0].view(np.float64), out[1].view(np.float64)), (parity, dagger)


@pytest.mark.parametrize("sloppy", ["f64", "f32", "f16", "bf16"])
@pytest.mark.parametrize("method", ["wilson_cg", "wilson_bicgstab"])
def test_split_solves(sloppy, method, monkeypatch):
    w = need_gpu()
    monkeypatch.setenv("WL_TUNE_FORCE", "11:64")
    L = (6, 4, 4, 10)
    U, eta = li.near_identity_links(L, 0.3, 63), li.gaussian_spinor(L, 64, nrhs=2)
    g = w.Gauge(L, to_dev(U))
    x = to_dev(np.zeros_like(eta))
    getattr(w, method)(g, to_dev(eta), x, 2, 0.12, 1e-10, 1000, sloppy, 12)
    psi = from_dev(x, eta.shape)
    g.close()
    r = eta - oracle.wilson(L, U, psi, 0.12)
    assert np.linalg.norm(r) <= 1.0001e-10 * np.linalg.norm(eta) * 2 ** 0.5


@pytest.mark.parametrize("L", [(2, 2, 2, 2), (4, 6, 2, 8)])
@pytest.mark.parametrize("prec,recon", CASES)
def test_split_clover_equals_per_site(L, prec, recon, monkeypatch):
    """A at the output site (the operator, both parities in one launch)."""
    w = need_gpu()
    U, psi = li.haar_links(L, 65), li.gaussian_spinor(L, 66, nrhs=2)
    for dagger in (0, 1):
        out = []
        for cfg in ("3:256", "11:64"):
            monkeypatch.setenv("WL_TUNE_FORCE", cfg)
            g = w.Gauge(L, to_dev(U))
            res = to_dev(np.full_like(psi, np.nan))
            w.wilson_clover_dslash(g, to_dev(psi), res, 2, 0.12, 1.3, dagger, prec, recon)
            out.append(from_dev(res, psi.shape))
            g.close()
        assert np.array_equal(out[0].view(np.float64), out[1].view(np.float64)), dagger


@pytest.mark.parametrize("sloppy", ["f64", "f32", "f16", "bf16"])
def test_split_clover_solves(sloppy, monkeypatch):
    """A and its inverse at the output sites (the solver's two hops)."""
    w = need_gpu()
    L = (6, 4, 4, 10)
    U, eta = li.near_identity_links(L, 0.3, 67), li.gaussian_spinor(L, 68)
    xs = []
    for cfg in ("3:256", "11:64"):
        monkeypatch.setenv("WL_TUNE_FORCE", cfg)
        for method in ("wilson_clover_cg", "wilson_clover_bicgstab"):
            g = w.Gauge(L, to_dev(U))
            x = to_dev(np.zeros_like(eta))
            getattr(w, method)(g, to_dev(eta), x, 1, 0.12, 1.0, 1e-11, 1000, sloppy, 12)
            xs.append(from_dev(x, eta.shape))
            g.close()
    # residual 1e-11 |eta|: solutions differ by at most 2e-11 |eta| / (smallest singular value of D > 0.02)
    for x in xs[1:]:
        assert np.linalg.norm(x - xs[0]) <= 1e-9 * np.linalg.norm(eta)
