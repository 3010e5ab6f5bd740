"""Forms of one solver step that must give the same bits: the solution updated in
each iteration and once for two, at chunk lengths that end in either; the FP64
residual rounded by its hop and stored and converted."""
import numpy as np
import pytest

import lattice_inputs as li
from tests.gpu_util import from_dev, need_gpu, to_dev

pytestmark = pytest.mark.gpu
SIZES = [(2, 2, 2, 4), (4, 6, 2, 8), (6, 4, 4, 10)]  # 16, 192 and 480 sites a parity


def solve(w, method, prec, recon, tol, maxiter, delta, csw=None):
    """The batch's solutions and iteration and update counts."""
    nrhs, kappa = [1, 3, 2], [0.12, 0.122, 0.1245]
    U = [li.near_identity_links(L, 0.3, 50 + i) for i, L in enumerate(SIZES)]
    eta = [li.gaussian_spinor(L, 60 + i, nrhs=n) for i, (L, n) in enumerate(zip(SIZES, nrhs))]
    eta[1][1] = 0  # a zero source is masked from the start
    g = [w.Gauge(L, to_dev(u)) for L, u in zip(SIZES, U)]
    x = [to_dev(np.zeros_like(e)) for e in eta]
    de = [to_dev(e) for e in eta]
    if method == "multi":
        info = w.wilson_cg_multi(g, de, x, nrhs, kappa, tol, maxiter, prec, recon, delta, check=False)[1]
    else:
        info = []
        for h, e, v, n, k in zip(g, de, x, nrhs, kappa):
            a = (h, e, v, n, k) + (() if csw is None else (csw,)) + (tol, maxiter, prec, recon, delta)
            info += getattr(w, method)(*a, check=False)[1]
    for h in g:
        h.close()
    return [from_dev(v, e.shape) for v, e in zip(x, eta)], [(i["iters"], i["reliable_updates"]) for i in info]


@pytest.mark.parametrize("method,csw", [("multi", None), ("wilson_cg", None), ("wilson_clover_cg", 1.0)])
@pytest.mark.parametrize("prec,recon", [("f64", 18), ("f32", 12), ("f16", 12), ("bf16", 12)])
def test_chunk_lengths_leave_the_same_bits(prec, recon, method, csw, monkeypatch):
    """Twelve iterations in chunks of one (x updated in each), and in chunks that end
    in a pair and in a single one, launched and replayed.  WL_TUNE=0: the six-launch
    iteration, with every launch in one configuration."""
    w = need_gpu()
    monkeypatch.setenv("WL_TUNE", "0")
    runs = {}
    for k in (1, 2, 3, 4, 6, 12):
        for graphs in "01":
            monkeypatch.setenv("WL_CHUNK", str(k))
            monkeypatch.setenv("WL_GRAPHS", graphs)
            runs[k, graphs] = solve(w, method, prec, recon, 1e-14, 12, 1e-9, csw)
    x, counts = runs[1, "0"]
    assert set(counts) == {(12, 1), (0, 0)} and counts.count((0, 0)) == 1, counts
    for key, (y, c) in runs.items():
        assert c == counts, key
        for a, b in zip(x, y):
            assert np.array_equal(a.view(np.float64), b.view(np.float64)), key


@pytest.mark.parametrize("k", [1, 2, 3, 5])
@pytest.mark.parametrize("prec,tol", [("f64", 1e-12), ("f32", 1e-5)])
def test_four_launch_iteration_at_every_chunk_end(prec, tol, k, monkeypatch):
    """The four-launch form closes each chunk with an update of x and p by itself."""
    w = need_gpu()
    monkeypatch.setenv("WL_CHUNK", str(k))
    a = solve(w, "multi", prec, 18, 1e-14, 10, 1e-9)
    monkeypatch.setenv("WL_TUNE", "0")
    b = solve(w, "multi", prec, 18, 1e-14, 10, 1e-9)
    assert a[1] == b[1] and {i for i, _ in a[1]} == {0, (10 + k - 1) // k * k}
    for x, y in zip(a[0], b[0]):
        assert np.linalg.norm(x - y) <= tol * np.linalg.norm(y)


@pytest.mark.parametrize("prec,recon,cfg", [(p, r, c) for p, r in [("f32", 18), ("f32", 12), ("f16", 12), ("bf16", 12)]
                                            for c in ("3:256", "0:64", "11:64") if p == "f32" or c != "11:64"])
@pytest.mark.parametrize("method,csw", [("multi", None), ("wilson_bicgstab", None), ("wilson_clover_cg", 1.0)])
def test_residual_rounded_in_the_hop(prec, recon, method, csw, cfg, monkeypatch):
    """(variant 11 rounds to FP32 only)"""
    w = need_gpu()
    monkeypatch.setenv("WL_TUNE_FORCE", cfg)
    runs = []
    for keep in "01":
        monkeypatch.setenv("WL_KEEP_RESIDUAL", keep)
        runs.append(solve(w, method, prec, recon, 1e-10, 500, 0.1, csw))
    assert runs[0][1] == runs[1][1] and max(u for _, u in runs[0][1]) >= 3
    for a, b in zip(runs[0][0], runs[1][0]):
        assert np.array_equal(a.view(np.float64), b.view(np.float64))
