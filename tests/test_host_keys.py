"""What the tuner's key and the plan index of a hop tell apart (CPU): a configuration found on one
set is used for every set of the same key, so sets whose candidates differ need
different keys.  Pencil blocks need the time extent to be a multiple of their
slices and time slices of whole waves, and some variants several right-hand sides
in a system: lattices of the same volume and batches of the same number of
vectors can differ in both."""
import ctypes
import os
import subprocess

import numpy as np
import pytest

HERE = os.path.dirname(os.path.abspath(__file__))
PKG = os.path.join(os.path.dirname(HERE), "paper_2001_05706_amd")


@pytest.fixture(scope="module")
def keys(tmp_path_factory):
    out = str(tmp_path_factory.mktemp("keys") / "libkeys.so")
    cmd = ["/opt/rocm/bin/hipcc", "--offload-arch=gfx950", "-O1", "-std=c++17", "-fPIC", "-shared", "-w",
           os.path.join(HERE, "host_keys.hip"), "-o", out, "-L" + PKG, "-l:libwilson.so", "-Wl,-rpath," + PKG]
    subprocess.run(cmd, check=True, capture_output=True)
    return ctypes.CDLL(out)


@pytest.fixture(scope="module")
def key(keys):
    lib = keys

    def of(*systems):
        L = np.array([s[0] for s in systems], dtype=np.int32)
        n = np.array([s[1] for s in systems], dtype=np.int32)
        buf = ctypes.create_string_buffer(1 << 16)
        assert lib.hop_key_of(len(systems), L.ctypes.data_as(ctypes.c_void_p), n.ctypes.data_as(ctypes.c_void_p), buf,
                              len(buf)) == 0
        return buf.value.decode()

    return of


@pytest.mark.parametrize("a,b", [
    # 8-slice pencils tile the first and not the second
    ([((32, 32, 36, 32), 1)], [((32, 32, 32, 36), 1)]),
    # slices of whole waves in the first only
    ([((16, 16, 16, 20), 1)], [((16, 16, 20, 16), 1)]),
    ([((8, 4, 4, 18), 1)], [((4, 4, 2, 72), 1)]),
    # the same vectors as right-hand sides of one system and as systems of one each
    ([((8, 8, 8, 16), 2)], [((8, 8, 8, 16), 1)] * 2),
    ([((8, 8, 8, 16), 3), ((4, 4, 4, 8), 1)], [((8, 8, 8, 16), 2), ((8, 8, 8, 16), 1), ((4, 4, 4, 8), 1)]),
])
def test_keys_differ(key, a, b):
    assert key(*a) != key(*b)


def test_keys_agree_for_the_same_shape(key):
    s = [((8, 8, 8, 16), 2), ((4, 4, 4, 8), 1)]
    assert key(*s) == key(*s)


@pytest.mark.parametrize("prec", range(4))
def test_plans_differ_where_only_variant_11_can_serve(keys, prec):
    """Of a D-slash call that reads the canonical input in the hop and one that packs it."""
    ids = [keys.plan_id_of(prec, nx, twin, direct) for nx in (0, 1) for twin in (0, 1) for direct in (0, 1)]
    assert len(set(ids)) == len(ids)
