"""The launch table, compiled for the host: a shape that a caller sets runs as
it was set, whatever the call asks for; a default read and set again is the
default; the defaults of calls with statuses, without a gradient or with Z are
adjusted."""
import ctypes
import os
import subprocess

import pytest

from paper_1807_08084_amd import _lib as L

HERE = os.path.dirname(os.path.abspath(__file__))
CALLS = {
    "inverse with statuses, large": ((6, L.F32, L.ADJUGATE, L.COMPENSATED),
                                     ("inv_det", (ctypes.c_int64(1 << 26), L.F32, L.ADJUGATE, L.COMPENSATED, 1))),
    "multilook with Z": ((2, L.F32, L.ADJUGATE, L.COMPENSATED), ("multilook", (L.F32, L.ADJUGATE, L.COMPENSATED, 4, 1))),
    "wishart forward, small": ((5, L.F32, 0, 0), ("wishart", (ctypes.c_int64(1 << 20), L.F32, 0))),
    "wishart forward, large": ((1, L.F64, 0, 0), ("wishart", (ctypes.c_int64(1 << 24), L.F64, 0))),
}


@pytest.fixture(scope="module")
def lib():
    so = os.path.join(HERE, "host", "liblaunch_host.so")
    subprocess.check_call(["g++", "-O2", "-std=c++17", "-fPIC", "-shared", "-o", so + ".tmp",
                           os.path.join(HERE, "host", "launch_host.cpp")])
    os.replace(so + ".tmp", so)
    return ctypes.CDLL(so)


def _get(lib, key):
    c = L.Launch()
    lib.host_get(*key, ctypes.byref(c))
    return c.as_dict()


def _run(lib, call):
    c = L.Launch()
    getattr(lib, "host_" + call[0])(*call[1], ctypes.byref(c))
    return c.as_dict()


@pytest.mark.parametrize("name", list(CALLS))
def test_a_set_shape_runs_as_set(lib, name):
    key, call = CALLS[name]
    default, adjusted = _get(lib, key), _run(lib, call)
    assert adjusted != default and dict(adjusted, blocks_per_cu=0) == dict(default, blocks_per_cu=0)
    for cfg in (dict(default, block=64, blocks_per_cu=default["blocks_per_cu"]), dict(default, blocks_per_cu=3),
                dict(default, blocks_per_cu=0), dict(default, blocks_per_cu=40)):
        lib.host_set(*key, ctypes.byref(L.Launch(**cfg)))
        assert _get(lib, key) == cfg and _run(lib, call) == cfg
    lib.host_set(*key, ctypes.byref(L.Launch(**default)))
    assert _get(lib, key) == default and _run(lib, call) == adjusted


def test_calls_without_an_adjustment_take_the_table(lib):
    for call, key in ((("inv_det", (ctypes.c_int64(1 << 26), L.F32, L.ADJUGATE, L.COMPENSATED, 0)), (6, L.F32, 0, 1)),
                      (("inv_det", (ctypes.c_int64(1 << 20), L.F32, L.ADJUGATE, L.COMPENSATED, 1)), (0, L.F32, 0, 1)),
                      (("inv_det", (ctypes.c_int64(1 << 26), L.F64, L.ADJUGATE, L.COMPENSATED, 1)), (6, L.F64, 0, 1)),
                      (("multilook", (L.F32, L.ADJUGATE, L.COMPENSATED, 3, 1)), (2, L.F32, 0, 1)),
                      (("multilook", (L.F32, L.ADJUGATE, L.COMPENSATED, 4, 0)), (2, L.F32, 0, 1)),
                      (("wishart", (ctypes.c_int64(1 << 20), L.F32, 1)), (5, L.F32, 0, 0))):
        assert _run(lib, call) == _get(lib, key)


@pytest.mark.parametrize("n,want_st,more", [(1 << 20, 1, 0), ((1 << 20) + 1, 1, 1), (1801 * 1799, 1, 1), ((1 << 22) - 1, 1, 1),
                                            (1 << 22, 1, 0), (1801 * 1799, 0, 0)])
def test_one_more_block_for_statuses_of_middle_sizes(lib, n, want_st, more):
    key = (0, L.F32, L.ADJUGATE, L.COMPENSATED)
    default = _get(lib, key)
    call = ("inv_det", (ctypes.c_int64(n),) + key[1:] + (want_st,))
    assert _run(lib, call) == dict(default, blocks_per_cu=default["blocks_per_cu"] + more)
    lib.host_set(*key, ctypes.byref(L.Launch(**dict(default, block=64))))
    assert _run(lib, call) == dict(default, block=64)
    lib.host_set(*key, ctypes.byref(L.Launch(**default)))


@pytest.mark.parametrize("dtype", [L.F32, L.F64])
def test_batch_of_likelihoods_alone(lib, dtype):
    key = (3, dtype, L.ADJUGATE, L.COMPENSATED)
    default = _get(lib, key)
    assert _run(lib, ("batch", key[1:] + (1,))) == default
    assert _run(lib, ("batch", key[1:] + (0,))) == dict(default, blocks_per_cu=2 * default["blocks_per_cu"])
    lib.host_set(*key, ctypes.byref(L.Launch(**dict(default, block=64))))
    assert _run(lib, ("batch", key[1:] + (0,))) == dict(default, block=64)
    lib.host_set(*key, ctypes.byref(L.Launch(**default)))
