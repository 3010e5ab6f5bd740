"""The four-launch CGNR iteration of small FP32 and FP64 sets: uneven batches on
lattices of less than one, one and several blocks of 64 sites reach the residual
the oracle confirms, in about the iterations of the six-launch form (which
WL_TUNE=0 runs), eager and replayed from a graph alike."""
import numpy as np
import pytest

import lattice_inputs as li
import oracle
from tests.gpu_util import from_dev, need_gpu, to_dev

pytestmark = pytest.mark.gpu
SIZES = [(2, 2, 2, 4), (4, 4, 4, 2), (4, 6, 2, 8), (6, 4, 4, 10)]  # 16, 64, 192, 480 sites a parity


@pytest.mark.parametrize("sloppy,recon", [("f64", 18), ("f64", 12), ("f32", 18), ("f32", 12)])
def test_small_batch(sloppy, recon, monkeypatch):
    w = need_gpu()
    nrhs = [1, 3, 2, 1]
    U = [li.near_identity_links(L, 0.3, 70 + i) for i, L in enumerate(SIZES)]
    eta = [li.gaussian_spinor(L, 80 + i, nrhs=n) for i, (L, n) in enumerate(zip(SIZES, nrhs))]
    eta[1][1] = 0  # a zero source is masked from the start
    runs = {}
    for name, env in (("graph", {}), ("eager", {"WL_GRAPHS": "0"}), ("six", {"WL_TUNE": "0"})):
        with monkeypatch.context() as m:
            for k, v in env.items():
                m.setenv(k, v)
            g = [w.Gauge(L, to_dev(u)) for L, u in zip(SIZES, U)]
            x = [to_dev(np.zeros_like(e)) for e in eta]
            _, info = w.wilson_cg_multi(g, [to_dev(e) for e in eta], x, nrhs, [0.12, 0.122, 0.12, 0.124], 1e-10, 1000,
                                        sloppy, recon)
            runs[name] = [from_dev(v, e.shape) for v, e in zip(x, eta)], info
            for h in g:
                h.close()
    for i, L in enumerate(SIZES):
        assert np.array_equal(runs["graph"][0][i], runs["eager"][0][i])
        for r in range(nrhs[i]):
            e, x = eta[i][r:r + 1], runs["graph"][0][i][r:r + 1]
            res = e - oracle.wilson(L, U[i], x, [0.12, 0.122, 0.12, 0.124][i])
            assert np.linalg.norm(res) <= 1.0001e-10 * np.linalg.norm(e)
    for a, b in zip(runs["graph"][1], runs["six"][1]):
        assert abs(a["iters"] - b["iters"]) <= 2 + b["iters"] // 10 and a["converged"] == b["converged"]


@pytest.mark.parametrize("sloppy,tol", [("f64", 1e-12), ("f32", 1e-5)])
@pytest.mark.parametrize("maxiter", [1, 2, 3, 6, 7])
def test_paired_solution_update(sloppy, tol, maxiter, monkeypatch):
    """A few iterations, odd and even, leave the solution that the four-launch form
    (which updates it in every iteration) leaves, to the rounding of the recurrence."""
    w = need_gpu()
    nrhs = [1, 3, 2, 1]
    kappa = [0.12, 0.122, 0.12, 0.124]
    eta = [li.gaussian_spinor(L, 80 + i, nrhs=n) for i, (L, n) in enumerate(zip(SIZES, nrhs))]
    eta[1][1] = 0  # a zero source is masked from the start
    runs = []
    for tune in ("1", "0"):
        with monkeypatch.context() as m:
            m.setenv("WL_TUNE", tune)
            g = [w.Gauge(L, to_dev(li.near_identity_links(L, 0.3, 70 + i))) for i, L in enumerate(SIZES)]
            x = [to_dev(np.zeros_like(e)) for e in eta]
            _, info = w.wilson_cg_multi(g, [to_dev(e) for e in eta], x, nrhs, kappa, 1e-14, maxiter, sloppy, 18,
                                        check=False)
            runs.append(([from_dev(v, e.shape) for v, e in zip(x, eta)], info))
            for h in g:
                h.close()
    assert [i["iters"] for i in runs[0][1]] == [i["iters"] for i in runs[1][1]]
    for a, b in zip(runs[0][0], runs[1][0]):
        assert np.linalg.norm(a - b) <= tol * np.linalg.norm(a)
