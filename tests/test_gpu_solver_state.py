"""What a solve takes and leaves: memory, hops, queued work."""
import numpy as np
import pytest

import lattice_inputs as li
import oracle
from tests.gpu_util import from_dev, need_gpu, to_dev

pytestmark = pytest.mark.gpu


def test_cgnr_needs_no_field_that_bicgstab_does_not():
    """CGNR's second direction lies in memory that the iterations leave idle."""
    import torch

    w = need_gpu()
    L = (24, 24, 24, 48)
    V = L[0] * L[1] * L[2] * L[3]
    g = w.Gauge(L, to_dev(li.near_identity_links(L, 0.3, 41)))
    gen = torch.Generator(device="cuda").manual_seed(42)
    eta = torch.randn(V * 24, generator=gen, dtype=torch.float64, device="cuda")
    x = torch.zeros_like(eta)
    solve = lambda f: (x.zero_(), f(g, eta, x, 1, 0.12, 1e-6, 200, "f64", 18))
    solve(w.wilson_bicgstab)
    free = torch.cuda.mem_get_info()[0]
    solve(w.wilson_cg)
    used = free - torch.cuda.mem_get_info()[0]
    g.close()
    # block maps, launch plans and graphs come to a few MiB; one field is 64
    assert used < V // 2 * 192 // 2


@pytest.mark.parametrize("sloppy", ["bf16", "f16", "f32"])
def test_hops_of_an_escalated_solve(sloppy):
    """Raising the sloppy precision costs the hops of its restart and no others: the
    FP64 residual of the update that found the stagnation is still there."""
    w = need_gpu()
    L = (8, 8, 8, 8)
    g = w.Gauge(L, to_dev(li.near_identity_links(L, 0.3, 1002)))
    eta = to_dev(li.gaussian_spinor(L, 2002))
    x = to_dev(np.zeros((1, 4096, 4, 3), dtype=complex))
    w.wl_prof_read()
    w.wl_prof_enable(True)
    try:
        _, info = w.wilson_cg(g, eta, x, 1, 0.1245, 1e-10, 5000, sloppy, 12, 0.9)
    finally:
        w.wl_prof_enable(False)
        launches = w.wl_prof_read()[0]
        g.close()
    info = info[0]
    assert info["precision_escalations"] > 0, info
    # b' and the first s = M^+ r; four an iteration; the FP64 residual and s an update;
    # s in the raised precision; odd sites and the true residual
    want = 1 + 2 + 4 * info["iters"] + 4 * info["reliable_updates"] + 2 * info["precision_escalations"] + 3
    assert launches == want, (launches, want, info)


@pytest.mark.parametrize("sloppy", ["bf16", "f16", "f32"])
def test_escalation_of_a_batch(sloppy):
    """Systems that stall at different times: the others are folded in and their
    residuals formed anew, and every later report is the one waited for."""
    w = need_gpu()
    Ls, nrhs, kappa = [(8, 8, 8, 8), (4, 6, 2, 8), (6, 4, 4, 10)], [1, 3, 2], [0.1245, 0.12, 0.122]
    U = [li.near_identity_links(L, 0.3, 1002 + i) for i, L in enumerate(Ls)]
    eta = [li.gaussian_spinor(L, 2002 + i, nrhs=n) for i, (L, n) in enumerate(zip(Ls, nrhs))]
    eta[1][1] = 0
    g = [w.Gauge(L, to_dev(u)) for L, u in zip(Ls, U)]
    x = [to_dev(np.zeros_like(e)) for e in eta]
    _, info = w.wilson_cg_multi(g, [to_dev(e) for e in eta], x, nrhs, kappa, 1e-10, 5000, sloppy, 12, 0.9)
    for h in g:
        h.close()
    assert info[0]["precision_escalations"] > 0
    for L, u, e, v, k in zip(Ls, U, eta, x, kappa):
        psi = from_dev(v, e.shape)
        for r in range(e.shape[0]):
            res = e[r:r + 1] - oracle.wilson(L, u, psi[r:r + 1], k)
            assert np.linalg.norm(res) <= 1.0001e-10 * np.linalg.norm(e[r:r + 1])


def test_a_refused_source_leaves_nothing_running():
    import torch

    w = need_gpu()
    L = (24, 24, 24, 32)
    V = L[0] * L[1] * L[2] * L[3]
    g = w.Gauge(L, to_dev(li.near_identity_links(L, 0.3, 45)))
    eta = torch.ones(4 * V * 24, dtype=torch.float64, device="cuda")
    x = torch.zeros_like(eta)
    busy = []
    eta[7] = float("nan")
    for _ in range(5):
        st, _ = w.wilson_cg(g, eta, x, 4, 0.12, 1e-8, 100, "f16", 12, check=False)
        busy.append(not torch.cuda.current_stream().query())
        assert st == 7  # WL_ERR_NONFINITE
    g.close()
    assert not any(busy)


@pytest.mark.parametrize("method,csw", [("wilson_cg", None), ("wilson_bicgstab", None), ("wilson_clover_cg", 1.0)])
@pytest.mark.parametrize("sloppy", ["f16", "bf16"])
def test_raise_to_a_precision_that_another_handle_has_tuned(sloppy, method, csw, monkeypatch):
    """The raised precision's configurations are known before this handle has met them:
    their block maps are made outside the capture of its chunks.  (A source of 1e30
    overflows FP16's and BF16's FP32 squares, which raises the precision.)"""
    w = need_gpu()
    L, nrhs = (8, 8, 8, 16), 9  # 576 blocks of 64 sites: tuned
    U, eta = to_dev(li.near_identity_links(L, 0.3, 46)), li.gaussian_spinor(L, 47, nrhs=nrhs)

    def solve(prec, scale):
        g, x = w.Gauge(L, U), to_dev(np.zeros_like(eta))
        a = (g, to_dev(eta * scale), x, nrhs, 0.12) + (() if csw is None else (csw,)) + (1e-10, 1000, prec, 12)
        _, info = getattr(w, method)(*a)
        g.close()
        return info

    for prec in ("f32", "f64"):
        assert all(i["converged"] for i in solve(prec, 1.0))
    monkeypatch.setenv("WL_TUNE_FORCE", "4:128:5")  # half precision only: its block maps are no other's
    info = solve(sloppy, 1e30)
    assert all(i["converged"] and i["precision_escalations"] >= 1 for i in info), info
