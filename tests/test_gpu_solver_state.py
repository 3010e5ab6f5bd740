"""What a solve takes and leaves: memory, hops, queued work."""
import numpy as np
import pytest

import lattice_inputs as li
from tests.gpu_util import need_gpu, to_dev

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
