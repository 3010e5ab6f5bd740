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
