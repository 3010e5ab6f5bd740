"""Launch plans and the calls that meet them in an unusual order."""
import numpy as np
import pytest

import lattice_inputs as li
from tests.gpu_util import from_dev, need_gpu, to_dev
from tests.test_gpu_dslash import CASES

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("prec,recon", CASES)
@pytest.mark.parametrize("parity", [0, -1])
def test_plan_of_a_packed_call_is_not_a_direct_calls(prec, recon, parity, monkeypatch):
    """A pinned configuration that is no candidate runs the tuner on a small set, and
    WL_TUNE=0 then takes what it found; without the settings the call reads the
    canonical field in the hop, which needs variant 11."""
    w = need_gpu()
    for L in [(2, 2, 2, 4), (4, 6, 2, 8), (6, 4, 4, 10), (8, 8, 8, 12)]:  # 1, 3, 8 and 48 blocks of 64 sites
        U, psi = li.haar_links(L, 31), li.gaussian_spinor(L, 32)
        g = w.Gauge(L, to_dev(U))
        din, out = to_dev(psi), []
        for env in ({"WL_TUNE_FORCE": "99:64"}, {"WL_TUNE": "0"}, {}):
            with monkeypatch.context() as m:
                for k, v in env.items():
                    m.setenv(k, v)
                o = to_dev(np.full_like(psi, np.nan))
                w.wilson_dslash(g, din, o, 1, 0.12, parity, 0, prec, recon)
                out.append(from_dev(o, psi.shape))
        g.close()
        assert np.array_equal(out[0], out[1]) and np.array_equal(out[0], out[2])


@pytest.mark.parametrize("prec,recon", [("f64", 18), ("f32", 12), ("bf16", 12)])
@pytest.mark.parametrize("L,nrhs", [((8, 8, 8, 16), 9), ((8, 8, 8, 16), 1)])  # 576 and 64 blocks of 64 sites
def test_other_parity_first_met_under_capture(L, nrhs, prec, recon):
    """A call with one output parity prepares the set for either: the other one can
    be captured, and its replays follow the input."""
    import torch

    w = need_gpu()
    g = w.Gauge(L, to_dev(li.haar_links(L, 34)))
    a, b = (to_dev(li.gaussian_spinor(L, 35 + i, nrhs=nrhs)) for i in range(2))
    inp, out, ref = a.clone(), torch.empty_like(a), torch.empty_like(a)
    w.wilson_dslash(g, inp, out, nrhs, 0.12, 0, 0, prec, recon)
    torch.cuda.synchronize()
    graph, s = torch.cuda.CUDAGraph(), torch.cuda.Stream()
    with torch.cuda.graph(graph, stream=s):
        w.wilson_dslash(g, inp, out, nrhs, 0.12, 1, 0, prec, recon)
    for src in (a, b, a):
        inp.copy_(src)
        out.fill_(float("nan"))
        graph.replay()
        torch.cuda.synchronize()
        w.wilson_dslash(g, inp, ref, nrhs, 0.12, 1, 0, prec, recon)
        torch.cuda.synchronize()
        assert torch.equal(out, ref)
    g.close()


def test_bench_dslash_times_the_hops_configuration(capfd, monkeypatch):
    """A small set's hop takes its variant without the tuner, and so does the
    measurement of it: nothing untimed goes into the tuner's table."""
    w = need_gpu()
    monkeypatch.setenv("WL_DEBUG", "1")
    L = (4, 4, 6, 10)
    g = w.Gauge(L, to_dev(li.haar_links(L, 33)))
    capfd.readouterr()
    for prec, recon in CASES:
        assert w.wl_bench_dslash(g, prec, recon, 1, 0, 1, 10) > 0
    g.close()
    assert "[wl tune]" not in capfd.readouterr().err


@pytest.mark.parametrize("L,nrhs,tuned", [((8, 8, 8, 8), 8, 0), ((8, 8, 8, 8), 9, 1), ((16, 16, 16, 16), 1, 1)])
def test_clover_operator_counts_both_parities(L, nrhs, tuned, capfd, monkeypatch):
    """256, 288 and 512 blocks of 64 sites a parity: one launch of both takes variant
    11 without the tuner up to 512 blocks in all; the Wilson operator counts one parity."""
    import torch

    w = need_gpu()
    monkeypatch.setenv("WL_DEBUG", "1")
    V = L[0] * L[1] * L[2] * L[3]
    gen = torch.Generator(device="cuda").manual_seed(37)
    psi = torch.randn(nrhs * V * 24, generator=gen, dtype=torch.float64, device="cuda")
    out = torch.empty_like(psi)
    g = w.Gauge(L, to_dev(li.near_identity_links(L, 0.3, 36)))
    capfd.readouterr()
    w.wilson_dslash(g, psi, out, nrhs, 0.12, -1, 0, "f16", 12)
    assert capfd.readouterr().err.count("[wl tune]") == 0
    w.wilson_clover_dslash(g, psi, out, nrhs, 0.12, 1.0, 0, "f16", 12)
    assert capfd.readouterr().err.count("[wl tune]") == tuned
    g.close()


def test_first_call_times_a_bounded_number_of_launches(capfd, monkeypatch):
    """The block orders and split forms of several right-hand sides make 288 candidates
    of a whole-lattice operator; where launches are long, the tuner tries them for the
    best few variants only.  Of at most 40 variants and block sizes 4 launches each, 7
    further forms of 6 of them and 16 again likewise, and 6 finalists in 3 trials of 9."""
    import re

    import torch

    w = need_gpu()
    monkeypatch.setenv("WL_DEBUG", "1")
    L, nrhs = (16, 16, 16, 20), 12
    V = 16 * 16 * 16 * 20
    gen = torch.Generator(device="cuda").manual_seed(38)
    psi = torch.randn(nrhs * V * 24, generator=gen, dtype=torch.float64, device="cuda")
    out = torch.empty_like(psi)
    g = w.Gauge(L, to_dev(li.near_identity_links(L, 0.3, 39)))
    capfd.readouterr()
    w.wilson_dslash(g, psi, out, nrhs, 0.12, -1, 0, "f32", 12)
    w.wilson_dslash(g, psi, out, nrhs, 0.12, 0, 0, "f32", 12)
    found = re.findall(r"\[wl tune\] .*; (\d+) candidates, (\d+) launches", capfd.readouterr().err)
    g.close()
    assert len(found) == 2 and max(int(c) for c, _ in found) >= 200
    assert all(int(n) <= 40 * 4 + 6 * 7 * 4 + 16 * 4 + 6 * 3 * 9 for _, n in found)


def hip():
    import ctypes

    h = ctypes.CDLL("libamdhip64.so")
    for f, a in (("hipStreamCreateWithFlags", [ctypes.c_void_p, ctypes.c_uint]),
                 ("hipStreamBeginCapture", [ctypes.c_void_p, ctypes.c_int]),
                 ("hipStreamEndCapture", [ctypes.c_void_p, ctypes.c_void_p]),
                 ("hipGraphDestroy", [ctypes.c_void_p]), ("hipStreamDestroy", [ctypes.c_void_p])):
        getattr(h, f).argtypes = a
    return h


class Capture:
    """A capture on a stream of its own (thread-local mode, as torch's graphs use at
    its strictest: nothing may be allocated or copied synchronously)."""

    def __init__(self):
        import ctypes

        self.h, self.s, self.g = hip(), ctypes.c_void_p(), ctypes.c_void_p()
        assert self.h.hipStreamCreateWithFlags(ctypes.byref(self.s), 1) == 0

    def __enter__(self):
        assert self.h.hipStreamBeginCapture(self.s, 1) == 0
        return self

    def __exit__(self, *a):
        import ctypes

        self.ended = self.h.hipStreamEndCapture(self.s, ctypes.byref(self.g))
        self.h.hipGetLastError()
        if self.g:
            self.h.hipGraphDestroy(self.g)
        self.h.hipStreamDestroy(self.s)


def test_a_failed_call_leaves_no_error_behind():
    """A call that cannot be captured (its fields do not exist yet) says so; the
    runtime's last error, which the next launch of any library would report, is clear."""
    w = need_gpu()
    L = (8, 8, 8, 16)
    psi = to_dev(li.gaussian_spinor(L, 51, nrhs=9))
    out = psi.clone()
    g = w.Gauge(L, to_dev(li.haar_links(L, 50)))
    with Capture() as c:
        with pytest.raises(w.WilsonError):
            w.wilson_dslash(g, psi, out, 9, 0.12, 0, 0, "f32", 12, stream=c.s.value)
        left = c.h.hipPeekAtLastError()
    w.wilson_dslash(g, psi, out, 9, 0.12, 0, 0, "f32", 12)
    g.close()
    assert left == 0


@pytest.mark.parametrize("clover", [False, True])
@pytest.mark.parametrize("prec,recon", [("f64", 18), ("f32", 12), ("f16", 12)])
def test_adjoint_first_met_under_capture(prec, recon, clover, monkeypatch):
    """A set that has run the operator can capture its adjoint, also in a configuration
    whose block map it has not made (here a pinned one; else one that another handle of
    the shape has tuned)."""
    import torch

    w = need_gpu()
    L, nrhs = (8, 8, 8, 16), 9
    g = w.Gauge(L, to_dev(li.haar_links(L, 52)))
    a, b = (to_dev(li.gaussian_spinor(L, 53 + i, nrhs=nrhs)) for i in range(2))
    inp, out, ref = a.clone(), torch.empty_like(a), torch.empty_like(a)

    def call(dagger, o):
        if clover:
            w.wilson_clover_dslash(g, inp, o, nrhs, 0.12, 1.0, dagger, prec, recon)
        else:
            w.wilson_dslash(g, inp, o, nrhs, 0.12, -1, dagger, prec, recon)

    call(0, out)
    torch.cuda.synchronize()
    graph, s = torch.cuda.CUDAGraph(), torch.cuda.Stream()
    monkeypatch.setenv("WL_TUNE_FORCE", "3:64:5")
    with torch.cuda.graph(graph, stream=s):
        call(1, out)
    monkeypatch.delenv("WL_TUNE_FORCE")
    for src in (a, b, a):
        inp.copy_(src)
        out.fill_(float("nan"))
        graph.replay()
        torch.cuda.synchronize()
        call(1, ref)
        torch.cuda.synchronize()
        assert torch.equal(out, ref)
    g.close()
