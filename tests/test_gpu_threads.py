"""Handles of different host threads: each solve on its own handle and stream, while
others set up, capture, solve and free theirs; and a capture of the caller's that is
open in another thread."""
import threading

import numpy as np
import pytest

import lattice_inputs as li
import oracle
from tests.gpu_util import from_dev, need_gpu, to_dev
from tests.test_gpu_plans import Capture

pytestmark = pytest.mark.gpu
SIZES = [(4, 4, 4, 8), (8, 8, 8, 8), (6, 4, 4, 10)]


def run(w, L, U, eta, prec, method, stream):
    """The operator and a solve on a new handle: (handle, D eta, x, status)."""
    import torch

    with torch.cuda.stream(stream):
        g = w.Gauge(L, U, stream=stream)
        out, x = torch.empty_like(eta), torch.zeros_like(eta)
        w.wilson_dslash(g, eta, out, 1, 0.12, -1, 0, prec, 12, stream=stream)
        st, _ = getattr(w, method)(g, eta, x, 1, 0.12, 1e-10, 500, prec, 12, check=False, stream=stream)
        stream.synchronize()
    return g, out, x, st


def test_threads_with_handles_of_their_own():
    import torch

    w = need_gpu()
    U = [li.near_identity_links(L, 0.3, 81 + i) for i, L in enumerate(SIZES)]
    eta = [li.gaussian_spinor(L, 84 + i) for i, L in enumerate(SIZES)]
    dU, de = [to_dev(u) for u in U], [to_dev(e) for e in eta]
    torch.cuda.synchronize()
    got, errors = [], []

    def work(t):
        stream = torch.cuda.Stream()
        for i in range(6):
            k, prec = (t + i) % 3, ("f64", "f32", "f16")[i % 3]
            try:
                g, out, x, st = run(w, SIZES[k], dU[k], de[k], prec, ("wilson_cg", "wilson_bicgstab")[i % 2], stream)
                got.append((k, prec, st, out, x))
                g.close()
            except Exception as e:  # reported by the main thread
                errors.append(e)
                return

    threads = [threading.Thread(target=work, args=(t,)) for t in range(3)]
    for t in threads:
        t.start()
    for t in threads:
        t.join()
    assert not errors, errors[0]
    assert len(got) == 18
    for k, prec, st, out, x in got:
        e = eta[k]
        res = e - oracle.wilson(SIZES[k], U[k], from_dev(x, e.shape), 0.12)
        assert st == 0 and np.linalg.norm(res) <= 1.0001e-10 * np.linalg.norm(e), (k, prec)
        ref = oracle.wilson(SIZES[k], U[k], e, 0.12)
        gate = {"f64": 1e-13, "f32": 1e-6, "f16": 3e-3}[prec]
        assert np.linalg.norm(from_dev(out, e.shape) - ref) <= gate * np.linalg.norm(ref), (k, prec)


def test_first_calls_beside_an_open_capture():
    """Setting up a handle, its fields and a solve in one thread leaves a capture open
    in another whole."""
    import torch

    w = need_gpu()
    L = (4, 4, 6, 8)
    U, eta = li.near_identity_links(L, 0.3, 87), li.gaussian_spinor(L, 88)
    dU, de, stream = to_dev(U), to_dev(eta), torch.cuda.Stream()
    torch.cuda.synchronize()
    res = []

    def work():
        try:
            for prec in ("f32", "f16"):
                res.append(run(w, L, dU, de, prec, "wilson_cg", stream))
        except Exception as e:  # reported by the main thread
            res.append(e)

    t = threading.Thread(target=work)
    with Capture() as c:
        t.start()
        t.join()
    for r in res:
        if isinstance(r, Exception):
            raise r
        g, out, x, st = r
        g.close()
        assert st == 0
    assert c.ended == 0
